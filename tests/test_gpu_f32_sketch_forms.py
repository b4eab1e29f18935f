"""The sketch of a float32 layer on both sides of the rule that chooses its form: tokens times rank next to the whole
workspace (the generic kernel) and at half of it (a stored S, several splits), both orientations of the small factor.

Bound: sums of n products in fp32 whose running sums are 512 long at most, 4 2^-24 sqrt(512); S is the device's own."""
import pytest

import plan_util as plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("n,channels,r,splits", [
    (16384, 512, 16, 0), (16381, 512, 24, 0), (8192, 256, 64, 0),
    (8190, 512, 24, 15), (24000, 1024, 64, 4), (2047, 256, 64, 1),
])
def test_sketch(acc, n, channels, r, splits, w_oi):
    import torch
    dev = "cuda:0"
    taken = plan.f32_sketch_splits(n, channels, r)
    assert (taken > 0) == (splits > 0) and abs(taken - splits) <= 1, taken
    g = torch.Generator(device=dev).manual_seed(n + r)
    X = torch.randn(n, channels, generator=g, device=dev)
    W = torch.randn(channels, 8, generator=g, device=dev)
    desc = acc.make_desc(n, channels, 8, r, seed=11, row_offset=40, io_dtype=acc.ACC_F32)
    S = torch.empty(n, r, device=dev)
    acc.acc_sketch_dump(desc, S)
    Y, Xs = torch.empty(n, 8, device=dev), torch.full((channels, r), 7.0, device=dev)
    print(f"f32 sketch {n} x {channels} rank {r}: {taken or 'generic'} w_oi={w_oi}", flush=True)
    acc.acc_linear_fwd(desc, X, W, Y, Xs, acc.alloc_workspace(desc, False, dev))
    # the small factor of a backward pass with `channels` outputs is the same product
    bdesc = acc.make_desc(n, 8, channels, r, seed=11, row_offset=40, io_dtype=acc.ACC_F32,
                          flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0)
    Wb = W.contiguous() if w_oi else W.T.contiguous()
    dX = torch.empty(n, 8, device=dev)
    Gr = torch.full((channels, r) if w_oi else (r, channels), 7.0, device=dev)
    acc.acc_linear_bwd(bdesc, X, Wb, None, dX, Gr, None, acc.alloc_workspace(bdesc, True, dev))
    want = X.double().T @ S.double()
    scale = want.square().mean().sqrt()
    for got in (Xs, Gr if w_oi else Gr.T):
        err = float((got.double() - want).square().mean().sqrt() / scale)
        worst = float((got.double() - want).abs().max() / scale)
        assert err <= 4 * 2.0 ** -24 * 512 ** 0.5 and worst <= 12 * 4 * 2.0 ** -24 * 512 ** 0.5, (err, worst)
