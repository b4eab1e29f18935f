"""The launch that factors and solves (ranks up to 128) over row counts: fewer rows than a work-group per 16 of them, a last block
of 16 rows that is partly empty, several row blocks per wave; and the two launches above rank 128.

X [n, d] holds scaled unit rows, so that Yr = X . Omega is exact in float32 and U [n, k] shows the factorisation alone, against
QR in 64 bits.  Bound: spread (sqrt(mean sigma^2 mean sigma^-2) of Yr's singular values) times k terms' rounding, as
test_gpu_qr_precision derives it, on single draws with a factor of 2."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


@pytest.mark.parametrize("n,k,d", [(64, 8, 64), (257, 40, 128), (4097, 128, 256), (33001, 72, 144), (66000, 24, 48), (8200, 200, 400)])
def test_rows(acc, n, k, d):
    import torch
    dev, u = "cuda:0", 2.0 ** -24
    X = torch.zeros(n, d, device=dev)
    i = torch.arange(n, device=dev)
    X[i, i % d] = 2.0 ** ((i // d) % 3).float()
    omega = torch.empty(d, k, device=dev)
    acc.acc_sketch_dump(acc.make_desc(d, 8, 8, k, seed=3, io_dtype=acc.ACC_F32), omega)
    desc = acc.make_desc(n, d, 8, k, seed=3, io_dtype=acc.ACC_F32)
    U, V, Y = torch.full((n, k), 7.0, device=dev), torch.empty(d, k, device=dev), torch.empty(n, 8, device=dev)
    print(f"n={n} k={k} d={d}", flush=True)
    acc.acc_linear_fwd_rsvd(desc, X, torch.zeros(d, 8, device=dev), Y, U, V, acc.alloc_workspace(desc, False, dev, rsvd=True))
    q, r = np.linalg.qr((X.double() @ omega.double()).cpu().numpy())
    q *= np.sign(np.diag(r))
    got = U.double().cpu().numpy()
    sigma2 = np.linalg.svd(r, compute_uv=False) ** 2
    bound = 2 * np.sqrt(np.mean(sigma2) * np.mean(1 / sigma2)) * (1.5 + k / (48 * d) ** 0.5)
    err, orth = np.linalg.norm(got - q) / np.linalg.norm(q), np.linalg.norm(got.T @ got - np.eye(k)) / np.sqrt(k)
    print(f"  |U - Q| {err / u:.2f} u of {bound:.2f}, |U^T U - I| {orth / u:.2f} u", flush=True)
    assert err <= bound * u and orth <= 6 * u
