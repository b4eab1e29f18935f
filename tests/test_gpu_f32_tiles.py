"""The float32 kernel at the edges of its tiles and K tiles: products in both weight layouts, the sketch with a stored S, and
the dense gradient in both result types.  Padding columns of every operand are NaN.

Bound: sums of K products in fp32, each partial sum rounded to 2^-24: 2^-24 sqrt(K) of the sum's own scale is expected,
four times that is allowed; the sketch adds its generator's 4e-6 of 1 / sqrt(r) per entry (measured, libm-grade)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import acc_oracle as orc
import plan_util as plan


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


def _padded(t, extra):
    import torch
    buf = torch.full((t.shape[0], t.shape[1] + extra), float("nan"), dtype=t.dtype, device=t.device)
    buf[:, :t.shape[1]] = t
    return buf


def _check(name, got, want, k, extra=0.0):
    scale = want.square().mean().sqrt()
    err = (got.double() - want).square().mean().sqrt() / scale
    worst = (got.double() - want).abs().max() / scale
    bound = 4 * 2.0 ** -24 * k ** 0.5 + extra
    print(f"  {name}: rms {float(err):.2e} worst {float(worst):.2e} bound {bound:.2e}", flush=True)
    assert err <= bound and worst <= 12 * bound, name    # 10^6 values: the largest lies about five sigma out


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("n,d_in,d_out,r,tiles", [   # tiles of Y, dX, dW and the forward sketch
    (1, 8, 8, 8, ["32x32"] * 4),                     # one chunk of everything
    (33, 40, 72, 16, ["32x32"] * 4),                 # second K tile of one or two chunks
    (300, 328, 296, 24, ["32x32"] * 4),              # K tiles more than stages, one token split, S beside nothing else
    (1030, 520, 1032, 40, ["64x32", "32x32", "32x32", "32x32"]),      # several token splits
    (2052, 1032, 2056, 64, ["64x32", "64x32", "64x32", "64x32"]),
    (1030, 1032, 1032, 1032, ["64x32"] * 4),         # 64 x 32 with both operands' rows contiguous, one split
    (776, 2048, 2048, 24, ["64x64", "64x64", "128x64", "32x32"]),     # dW: one K tile of a ring of three
    (2044, 2040, 2040, 40, ["128x64", "128x64", "128x64", "32x32"]),  # K ends inside a K tile
    (300, 2040, 2040, 2040, ["32x32", "32x32", "128x64", "128x64"]),  # 128 x 64 with both operands' rows contiguous
    (2330, 1480, 2504, 24, ["128x64", "128x64", "128x64", "64x32"]),  # Y: three 128 x 64 tiles to a compute unit
])
def test_layer(acc, n, d_in, d_out, r, tiles, out_in):
    import torch
    splits = plan.f32_sketch_splits(n, d_in, r)
    assert splits > 0 and tiles == [plan.f32_tile(n, d_out), plan.f32_tile(n, d_in), plan.f32_tile(d_in, d_out),
                                    plan.f32_tile(d_in, r, splits)]
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(n)
    X, dY = torch.randn(n, d_in, generator=g, device=dev), torch.randn(n, d_out, generator=g, device=dev)
    W = torch.randn(d_in, d_out, generator=g, device=dev)
    Wl = W.T.contiguous() if out_in else W
    Xp, Wp, dYp = _padded(X, 8), _padded(Wl, 16), _padded(dY, 24)
    S = torch.from_numpy(orc.sketch_matrix(5, n, r, 400)).to(dev)
    Xd, Wd, dYd = X.double(), W.double(), dY.double()
    want_xs, want_gr = Xd.T @ S, S.T @ dYd
    print(f"f32 layer {n} x {d_in} x {d_out} r={r} out_in={out_in}", flush=True)
    for code, dt in ((acc.ACC_F32, torch.float32), (acc.ACC_BF16, torch.bfloat16)):     # type of the dense gradient
        desc = acc.make_desc(n, d_in, d_out, r, seed=5, row_offset=400, io_dtype=acc.ACC_F32, dw_dtype=code, ldx=d_in + 8,
                             ldw=Wp.shape[1], ldy=d_out + 24, flags=acc.ACC_FLAG_W_OUT_IN if out_in else 0)
        Y, dX = torch.full_like(dYp, 7.0), torch.full_like(Xp, 7.0)
        Xs = torch.full((d_in, r), 7.0, device=dev)
        Gr = torch.full((d_out, r) if out_in else (r, d_out), 7.0, device=dev)
        dW = torch.full((d_out, d_in) if out_in else (d_in, d_out), 7.0, device=dev, dtype=dt)
        acc.acc_linear_fwd(desc, Xp, Wp, Y, Xs, acc.alloc_workspace(desc, False, dev))
        acc.acc_linear_bwd(desc, dYp, Wp, Xs, dX, Gr, dW, acc.alloc_workspace(desc, True, dev))
        torch.cuda.synchronize()
        assert torch.all(Y[:, d_out:] == 7.0) and torch.all(dX[:, d_in:] == 7.0)
        _check("Y", Y[:, :d_out], Xd @ Wd, d_in)
        _check("dX", dX[:, :d_in], dYd @ Wd.T, d_out)
        _check("Xs", Xs, want_xs, n, 4e-6)
        _check("Gr", Gr, want_gr.T if out_in else want_gr, n, 4e-6)
        left, right = Xs.double(), (Gr.T if out_in else Gr).double()   # the product of the factors as they were stored
        want = (left @ right).T if out_in else left @ right
        _check("dW", dW, want, r, 0.0 if dt == torch.float32 else 2.0 ** -9)
