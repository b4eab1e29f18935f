"""The Cholesky QR at the edges of its 16-column blocks and of its one-launch size (256), through the projector refresh in
float32: ranks that end inside a block, and factors whose rank ends inside one.

Bound: the basis inherits the conditioning of Yp = left . (Gr . Omega), so cond(Yp) times 1e-5 (float32 products of a few
hundred terms, normals accurate to 4e-6), evaluated from the oracle's Yp."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import acc_oracle as orc
import gpu_util as gu


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


def _projector(acc, left, gr, k, seed):
    import torch
    dev = "cuda:0"
    d_in, r = left.shape
    desc = acc.make_desc(1, d_in, gr.shape[1], r, seed=seed, io_dtype=acc.ACC_F32)
    P = torch.full((d_in, k), 7.0, device=dev)
    print(f"projector {d_in} x {gr.shape[1]} r={r} k={k}", flush=True)
    acc.acc_lowrank_projector(desc, k, acc.to_device(left, dev), acc.to_device(gr, dev), P,
                              acc.alloc_lowrank_workspace(desc, k, dev))
    torch.cuda.synchronize()
    return acc.to_host_f64(P)


@pytest.mark.parametrize("k", [8, 24, 64, 72, 128, 136, 256, 264, 512])
def test_basis(acc, k):
    rng = np.random.default_rng(k)
    d_in, d_out, r = 1208, 328 if k < 300 else 1032, max(k, 32)
    left = rng.standard_normal((d_in, r), dtype=np.float32)
    gr = rng.standard_normal((r, d_out), dtype=np.float32)
    got = _projector(acc, left, gr, k, 3)
    lo, go = left.astype(np.float64), gr.astype(np.float64)
    want = orc.gradient_projector(lo, go, 3, k)
    cond = np.linalg.cond(lo @ (go @ orc.range_finder_matrix(3, d_out, k)))
    err, orth = gu.rel(got, want), np.linalg.norm(got.T @ got - np.eye(k))
    print(f"  rel {err:.2e} cond {cond:.1f} |P^T P - I| {orth:.2e}", flush=True)
    assert err <= 1e-5 * cond and orth <= 1e-6 * k


@pytest.mark.parametrize("k,rank", [(24, 10), (72, 5), (136, 40), (264, 40), (320, 20)])
def test_dependent_columns_come_out_as_zero(acc, k, rank):
    """left = A . B of rank `rank` < k, small integers, so that left's rank is exact: the first `rank` columns of P are the
    basis of the range, the others zero.  Yp = left . (Gr . Omega) is rounded, so a dependent column keeps about 2^-24 of its
    size, which the second pass would pick up where few pivots separate it from the cut; the ranks stay clear of that."""
    rng = np.random.default_rng(rank)
    d_in, d_out, r = 1000, 296, 320
    A = rng.integers(-2, 3, (d_in, rank)).astype(np.float32)
    B = rng.integers(-1, 2, (rank, r)).astype(np.float32)
    left = A @ B
    gr = rng.standard_normal((r, d_out), dtype=np.float32)
    got = _projector(acc, left, gr, k, 4)
    norms = np.linalg.norm(got, axis=0)
    assert np.all(np.abs(norms[:rank] - 1) < 1e-4) and np.all(norms[rank:] == 0), norms[rank - 2:rank + 3]
    q = np.linalg.qr(A.astype(np.float64))[0]
    out = got[:, :rank] - q @ (q.T @ got[:, :rank])       # nothing outside range(A)
    assert np.linalg.norm(out) <= 1e-3 * np.sqrt(rank)
