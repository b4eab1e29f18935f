"""How long the running sums of the skinny split products are (the small factor of the RSVD backward pass, Gr = U^T . dY):
dY is one except for 2^30 in one row and -2^30 in another.  Additions of a matrix instruction's 32 ones to a float32 sum of
that size are lost, so a result tells how many elements share a running sum with the two large ones: at most 256 each.  All
sums of 256 and of splits are multiples of 128, the spacing of floats at 2^30, and add up exactly."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("n,d_in,d_out,k", [(16384, 3072, 3072, 32), (4096, 2048, 2048, 128), (2048, 512, 4096, 256)])
def test_running_sums_are_256_elements_long(acc, n, d_in, d_out, k, w_oi):
    import torch
    dev, big = "cuda:0", 2.0 ** 30
    first = [0, 300, n // 2 - 1, n // 3]
    dY = torch.ones(n, d_out, device=dev, dtype=torch.bfloat16)
    for c, p in enumerate(first):
        dY[p, c::4] = big
        dY[n - 1 - p, c::4] = -big
    U = torch.ones(n, k, device=dev, dtype=torch.bfloat16)
    W = torch.zeros(*((d_out, d_in) if w_oi else (d_in, d_out)), device=dev, dtype=torch.bfloat16)
    desc = acc.make_desc(n, d_in, d_out, k, io_dtype=acc.ACC_BF16, flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0)
    dX = torch.empty(n, d_in, device=dev, dtype=torch.bfloat16)
    Gr = torch.full((d_out, k) if w_oi else (k, d_out), 7.0, device=dev, dtype=torch.bfloat16)
    print(f"split sums {n} x {d_out} rank {k} w_oi={w_oi}", flush=True)
    acc.acc_linear_bwd_rsvd(desc, dY, W, U, None, dX, Gr, None, acc.alloc_workspace(desc, True, dev, rsvd=True))
    got = (Gr if w_oi else Gr.T).float().cpu()          # [d_out, k]
    assert torch.all(got <= n) and torch.all(got >= (n - 2 * 256) * (1 - 2.0 ** -8)), (float(got.min()), float(got.max()), n)
