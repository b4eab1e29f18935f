"""How close the Cholesky QR itself is to 64 bits, at the sizes where its sums get long: X holds scaled unit rows, so that
Yr = X . Omega is exact in float32 and U [n, k] (float32 factors) shows the factorisation's rounding alone, against QR in
64 bits of the Omega that the device made.

Bounds, with u = 2^-24, medians over six draws.  |U^T U - I| / sqrt(k): a column's scale is 1 / sqrt of its Gram entry; that sum
rounds at four levels (32 rows, their sums, the splits, the tree of those) and its root, reciprocal and product once each:
about 2 u expected, 3 u allowed.  |U - Q| / |Q|: an entry takes about 1.5 roundings at its own size; the sum it is
reduced by has k products in two chains, four products an addition, and reaches sqrt(k / d) of the entry, so its additions
round to k / sqrt(48 d) u; both are spread by R^-1, sqrt(mean sigma^2 mean sigma^-2) of the singular values sigma."""
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


@pytest.mark.parametrize("k,d", [(8, 8), (8, 64), (16, 128), (32, 256), (64, 128), (96, 192), (128, 1024), (192, 200),
                                 (256, 512), (256, 2048), (264, 528), (512, 1024)])
def test_rounding_of_the_factorisation(acc, k, d):
    import torch
    dev, u = "cuda:0", 2.0 ** -24
    n = max(d, -(-256 // d) * d)
    X = torch.zeros(n, d, device=dev)
    i = torch.arange(n, device=dev)
    X[i, i % d] = 2.0 ** ((i // d) % 3).float()
    orth, err, spreads = [], [], []
    for seed in range(1, 7):
        omega = torch.empty(d, k, device=dev)
        acc.acc_sketch_dump(acc.make_desc(d, 8, 8, k, seed=seed, io_dtype=acc.ACC_F32), omega)
        desc = acc.make_desc(n, d, 8, k, seed=seed, io_dtype=acc.ACC_F32)
        U, V = torch.empty(n, k, device=dev), torch.empty(d, k, device=dev)
        Y = torch.empty(n, 8, device=dev)
        acc.acc_linear_fwd_rsvd(desc, X, torch.zeros(d, 8, device=dev), Y, U, V, acc.alloc_workspace(desc, False, dev, rsvd=True))
        q, r = np.linalg.qr((X.double() @ omega.double()).cpu().numpy())
        q *= np.sign(np.diag(r))
        got = U.double().cpu().numpy()
        orth.append(np.linalg.norm(got.T @ got - np.eye(k)) / np.sqrt(k))
        err.append(np.linalg.norm(got - q) / np.linalg.norm(q))
        sigma2 = np.linalg.svd(r, compute_uv=False) ** 2
        spreads.append(np.sqrt(np.mean(sigma2) * np.mean(1 / sigma2)))
    o, e, spread = (float(np.median(v)) for v in (orth, err, spreads))
    bound = spread * (1.5 + k / (48 * d) ** 0.5)
    print(f"k={k} d={d} |U^T U - I| {o / u:.2f} u, |U - Q| {e / u:.2f} u of {bound:.2f}", flush=True)
    assert o <= 3 * u and e <= bound * u
