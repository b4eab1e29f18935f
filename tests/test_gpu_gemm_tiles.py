"""The exact products at the edges of their kernels' tiles and K tiles, one shape per kernel of the dispatch.

The contraction length is no multiple of 64, so the last K tile is partly empty; X and W sit in wider rows whose padding
is NaN, so a product that reads past K, or multiplies a zero by what lies there, shows.  Bound: the operands are exact
bfloat16 and the output is rounded once, 2^-9 per element at most; the fp32 sums add 1e-5 at these lengths."""
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


# (rows, columns, contraction): the tile the dispatch takes, and what is at an edge there
SHAPES = [
    (1, 8, 8),            # 64 x 64, less than one K tile
    (65, 72, 72),         # 64 x 64, one row and one chunk into the second tile, second K tile of one chunk
    (200, 520, 456),      # 64 x 64, more K tiles than stages
    (1400, 1032, 1000),   # 128 x 64
    (1053, 3048, 1592),   # 128 x 128, one round of tiles
    (2050, 3080, 1000),   # 128 x 128, several tiles per compute unit
    (1100, 5000, 2000),   # 192 x 128, one round of tiles
    (4000, 2056, 392),    # 192 x 128, several tiles per compute unit
    (4090, 3064, 392),    # 256 x 192, one round of tiles
    (8200, 4104, 136),    # 256 x 256, three K tiles, several tiles per work-group
    (600, 18008, 136),    # 256 x 256, three rows of tiles
]


def _padded(t, extra):
    import torch
    buf = torch.full((t.shape[0], t.shape[1] + extra), float("nan"), dtype=t.dtype, device=t.device)
    buf[:, :t.shape[1]] = t
    return buf


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_ragged_contraction(acc, m, n, k, out_in):
    import torch
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
    """dW = Xs.Gr on the short-contraction kernel (one round of tiles) and on the tiled ones, written and accumulated;
    the factor's padding columns are NaN."""
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
