"""The launch that a small float32 layer's exact product shares with its sketch, at the edges of its 32 x 32 tiles: remainders in
every dimension, one and several token splits (their partial products lie behind S and are folded), both weight orientations,
padded rows, a bfloat16 factor, the product's work-groups in front of the sketch's (where its contraction is longer than a split)
and behind them; and layers beyond it.

Bound: fp32 sums of 256 products, and of at most four of those, 4 2^-24 sqrt(512); a bfloat16 factor rounds once, 2^-8."""
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


# fwd, bwd: token splits of the sketch that shares a launch with the pass's exact product, 0 where it shares none
@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("n,d_in,d_out,r,pad,bf16_factor,fwd,bwd", [
    (256, 256, 512, 16, 0, False, 1, 1), (33, 40, 264, 8, 0, False, 1, 1), (257, 136, 136, 40, 8, False, 1, 1), (1, 8, 8, 8, 0, False, 1, 1),
    (257, 520, 136, 24, 16, True, 1, 0), (513, 136, 264, 24, 8, True, 0, 1),   # a bfloat16 factor is folded from one split too
    (1500, 512, 512, 16, 0, False, 3, 3), (900, 776, 712, 40, 8, False, 2, 2), (900, 776, 712, 40, 0, True, 2, 2),
    (1030, 520, 488, 24, 16, True, 3, 2), (2624, 384, 264, 64, 0, False, 4, 0), (700, 1000, 904, 256, 8, False, 1, 0), (2624, 264, 384, 64, 8, True, 0, 4),
    (33, 40, 24, 8, 0, False, 1, 0), (700, 64, 96, 32, 0, False, 0, 0), (2048, 1024, 1032, 64, 0, False, 0, 0),
])
def test_layer(acc, n, d_in, d_out, r, pad, bf16_factor, fwd, bwd, w_oi):
    import torch
    dev = "cuda:0"
    assert (plan.f32_pair(n, d_in, d_out, r, not bf16_factor), plan.f32_pair(n, d_out, d_in, r, not bf16_factor)) == (fwd, bwd)
    g = torch.Generator(device=dev).manual_seed(n + r)
    rand = lambda rows, cols, ld: torch.randn(rows, ld, generator=g, device=dev)[:, :cols]   # padded rows hold other values
    X, dY = rand(n, d_in, d_in + pad), rand(n, d_out, d_out + pad)
    W = rand(*((d_out, d_in, d_in + pad) if w_oi else (d_in, d_out, d_out + pad)))
    flags = acc.ACC_FLAG_W_OUT_IN if w_oi else 0
    desc = acc.make_desc(n, d_in, d_out, r, seed=11, row_offset=40, io_dtype=acc.ACC_F32, flags=flags, ldx=d_in + pad, ldy=d_out + pad,
                         ldw=W.stride(0), factor_dtype=acc.ACC_BF16 if bf16_factor else acc.ACC_F32)
    S = torch.empty(n, r, device=dev)
    acc.acc_sketch_dump(desc, S)
    ft = torch.bfloat16 if bf16_factor else torch.float32
    Y, dX = torch.full((n, d_out + pad), 7.0, device=dev), torch.full((n, d_in + pad), 7.0, device=dev)
    Xs = torch.full((d_in, r), 7.0, device=dev, dtype=ft)
    Gr = torch.full((d_out, r) if w_oi else (r, d_out), 7.0, device=dev, dtype=ft)
    print(f"f32 layer {n} x {d_in} x {d_out} rank {r} pad {pad} w_oi={w_oi}", flush=True)
    acc.acc_linear_fwd(desc, X, W, Y, Xs, acc.alloc_workspace(desc, False, dev))
    acc.acc_linear_bwd(desc, dY, W, Xs, dX, Gr, None, acc.alloc_workspace(desc, True, dev))
    Wd, Sd = (W.T if w_oi else W).double(), S.double()
    assert bool((Y[:, d_out:] == 7.0).all()) and bool((dX[:, d_in:] == 7.0).all())   # the gap between rows is the caller's
    tol = 4 * 2.0 ** -24 * 512 ** 0.5
    for name, got, want in (("Y", Y[:, :d_out], X.double() @ Wd), ("Xs", Xs, X.double().T @ Sd), ("dX", dX[:, :d_in], dY.double() @ Wd.T),
                            ("Gr", Gr if not w_oi else Gr.T, Sd.T @ dY.double())):
        bound = tol + (2.0 ** -8 if bf16_factor and name in ("Xs", "Gr") else 0)
        err = float((got.double() - want).norm() / want.norm())
        worst = float((got.double() - want).abs().max() / want.square().mean().sqrt())
        assert err <= bound and worst <= 12 * bound, (name, err, worst)
