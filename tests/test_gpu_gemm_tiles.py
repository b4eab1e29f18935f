"""The exact products at the edges of their kernels' tiles and K tiles, one shape per kernel of the dispatch.

The contraction length is no multiple of 64, so the last K tile is partly empty; X and W sit in wider rows whose padding
is NaN, so a product that reads past K, or multiplies a zero by what lies there, shows.  Bound: the operands are exact
bfloat16 and the output is rounded once, half a unit in the last place, 2^-8 of the element at most; the fp32 sums add 1e-5
at these lengths."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import plan_util as plan


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


# rows, columns, contraction, the tile the dispatch takes and whether it is one round of the chip; what is at an edge there
SHAPES = [
    (1, 8, 8, "64x64", True),               # less than one K tile
    (65, 72, 72, "64x64", True),            # one row and one chunk into the second tile, second K tile of one chunk
    (200, 520, 456, "64x64", True),         # more K tiles than stages
    (1400, 1032, 1000, "128x64", True),
    (1053, 3048, 1592, "128x128", True),
    (2050, 3080, 1000, "128x128", False),
    (1100, 5000, 2000, "192x128", True),
    (4000, 2056, 392, "192x128", False),
    (4090, 3064, 392, "256x192", True),
    (8200, 4104, 136, "256x256", False),    # three K tiles, several tiles per work-group
    (600, 18008, 136, "256x256", True),     # three rows of tiles
]


def _padded(t, extra):
    import torch
    buf = torch.full((t.shape[0], t.shape[1] + extra), float("nan"), dtype=t.dtype, device=t.device)
    buf[:, :t.shape[1]] = t
    return buf


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("m,n,k,tile,one_round", SHAPES)
def test_ragged_contraction(acc, m, n, k, tile, one_round, out_in):
    import torch
    assert plan.gemm_tile(m, n, k) == (tile, one_round)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    X = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    W = (torch.randn(k, n, generator=g, device="cuda") * 0.02).bfloat16()
    Xp, Wp = _padded(X, 8), _padded(W.T.contiguous() if out_in else W, 16)
    Y = torch.full((m, n + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    desc = acc.make_desc(m, k, n, 8, ldx=Xp.shape[1], ldw=Wp.shape[1], ldy=Y.shape[1],
                         flags=acc.ACC_FLAG_SKIP_SKETCH | (acc.ACC_FLAG_W_OUT_IN if out_in else 0))
    print(f"exact product {m} x {n} x {k} out_in={out_in}", flush=True)
    acc.acc_linear_fwd(desc, Xp, Wp, Y, None, None)
    got = Y.cpu()
    assert torch.all(got[:, n:] == 7.0)                     # padding columns untouched
    want = X.double().cpu().numpy() @ W.double().cpu().numpy() if m * n * k < 1 << 30 else (X.double() @ W.double()).cpu().numpy()
    err = np.abs(got[:, :n].double().numpy() - want)
    scale = np.sqrt(np.mean(want * want))
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + 1e-5 * scale), float(np.nanmax(err))


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("r", [8, 40, 72, 136, 200])
def test_dense_gradient_at_ragged_ranks(acc, r, out_in):
    """dW = Xs.Gr of a small and of a large output, written and accumulated in float; the factor's padding columns are NaN."""
    import torch
    for d_in, d_out in ((200, 392), (4104, 3080)):
        g = torch.Generator(device="cuda").manual_seed(r + d_in)
        Xs = torch.randn(d_in, r, generator=g, device="cuda").bfloat16()
        Gr = (torch.randn(r, d_out, generator=g, device="cuda") * 0.01).bfloat16()
        Xsp = _padded(Xs, 8)
        Grp = _padded(Gr.T.contiguous(), 8) if out_in else Gr
        want = Xs.double() @ Gr.double()
        want = want.T if out_in else want
        dW = torch.full(tuple(want.shape), 7.0, dtype=torch.float32, device="cuda")
        flags = acc.ACC_FLAG_W_OUT_IN if out_in else 0
        print(f"dense gradient {d_in} x {d_out} r={r} out_in={out_in}", flush=True)
        for passes in (1, 2):
            desc = acc.make_desc(1, d_in, d_out, r, ldf=r + 8, dw_dtype=acc.ACC_F32,
                                 flags=flags | (acc.ACC_FLAG_DW_ACCUMULATE if passes == 2 else 0))
            acc.acc_linear_dw(desc, Xsp, Grp, dW)
            err = (dW.double() - passes * want).abs().max()
            assert err <= 1e-5 * want.square().mean().sqrt(), (passes, float(err))  # fp32 sums of r <= 200 exact products


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("d_in,d_out,r,written,added,added_f32", [   # the kernel of each form; a float result is written as a bfloat16 one
    (3264, 3080, 40, "192x128", "128x64", "64x64"),
    (3504, 3104, 200, "192x128", "128x64", "64x64"),
    (520, 1032, 1096, "64x64", "64x64", "64x64"),
    (1400, 1032, 1032, "128x64", "128x64", "128x64"),
    (1056, 3048, 1592, "128x128", "128x128", "128x128"),
    (4096, 3072, 1032, "256x192", "256x192", "256x192"),
])
def test_dense_gradient_on_the_ring_kernel(acc, d_in, d_out, r, written, added, added_f32, out_in):
    """dW written and accumulated, in float and in bfloat16; the factor's padding columns are NaN, dW's neighbours stay."""
    import torch
    M, N = (d_out, d_in) if out_in else (d_in, d_out)
    taken = [plan.factor_tile(M, N, r, bf16_c, sums) for sums in (False, True) for bf16_c in (True, False)]
    assert out_in or taken == [written, written, added, added_f32], taken
    g = torch.Generator(device="cuda").manual_seed(r + d_in)
    Xs = torch.randn(d_in, r, generator=g, device="cuda").bfloat16()
    Gr = (torch.randn(r, d_out, generator=g, device="cuda") * 0.01).bfloat16()
    Xsp = _padded(Xs, 8)
    Grp = _padded(Gr.T.contiguous(), 8) if out_in else Gr
    want = Xs.double() @ Gr.double()
    want = want.T if out_in else want
    scale = want.square().mean().sqrt()
    print(f"ring dense gradient {d_in} x {d_out} r={r} out_in={out_in}", flush=True)
    for code, dt in ((acc.ACC_F32, torch.float32), (acc.ACC_BF16, torch.bfloat16)):
        buf = torch.full((M + 2, N), 7.0, dtype=dt, device="cuda")      # a row of guard on either side
        dW = buf[1:M + 1]
        exact = torch.zeros_like(want)
        for flag in (0, acc.ACC_FLAG_DW_ACCUMULATE, acc.ACC_FLAG_DW_ACCUMULATE):
            desc = acc.make_desc(1, d_in, d_out, r, ldf=r + 8, dw_dtype=code,
                                 flags=flag | (acc.ACC_FLAG_W_OUT_IN if out_in else 0))
            before = dW.double() if flag else torch.zeros_like(want)
            acc.acc_linear_dw(desc, Xsp, Grp, dW)
            exact = before + want
            allowed = 1e-5 * scale + (2.0 ** -8 * exact.abs() if dt == torch.bfloat16 else 1e-6 * exact.abs())
            assert torch.all((dW.double() - exact).abs() <= allowed), (dt, flag)
        assert torch.all(buf[0] == 7.0) and torch.all(buf[M + 1] == 7.0)
