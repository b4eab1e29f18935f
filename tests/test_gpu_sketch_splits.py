"""The bfloat16 sketch with bfloat16 factors, whose slabs and token splits pick_sketch_split chooses: ragged last slab, ragged last
split, surplus sketch columns, padded rows, both orientations, against a product in 64 bits with the device's own S.

Bound: one rounding to bfloat16, half a unit of 2^-8 of the value, and fp32 running sums of at most 4096 tokens and their sum,
4 2^-24 sqrt(4096) of the root mean square; 12 times that for the largest of many entries."""
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


@pytest.mark.parametrize("n,channels,r,pad,slab", [
    (300, 3064, 256, 0, 128), (601, 2056, 200, 8, 128), (1030, 520, 72, 0, 128),
    (4095, 4088, 128, 0, 256), (2050, 4096, 232, 16, 256), (8190, 2056, 128, 0, 256),
    (4097, 8184, 256, 8, 512), (8190, 3080, 200, 8, 512), (31, 264, 24, 0, 128),
])
def test_sketch(acc, n, channels, r, pad, slab):
    import torch
    most = max(1, min(256 // (-(-channels // 512) * -(-r // 64)), -(-n // 256), 64))
    assert plan.sketch_split(n, channels, r, most)[0] == slab
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(n + r)
    ld = channels + pad
    X = torch.randn(n, ld, generator=g, device=dev).bfloat16()[:, :channels]
    W = torch.randn(channels, 64, generator=g, device=dev).bfloat16()
    kw = dict(seed=11, row_offset=40)
    desc = acc.make_desc(n, channels, 64, r, ldx=ld, **kw)
    S = torch.empty(n, r, device=dev)
    acc.acc_sketch_dump(desc, S)
    Y, Xs = torch.empty(n, 64, device=dev, dtype=torch.bfloat16), torch.full((channels, r), 7.0, device=dev).bfloat16()
    print(f"sketch {n} x {channels} rank {r}", flush=True)
    acc.acc_linear_fwd(desc, X, W, Y, Xs, acc.alloc_workspace(desc, False, dev))
    got = [Xs]
    for w_oi in (False, True):   # the small factor of a backward pass with `channels` outputs is the same product
        bdesc = acc.make_desc(n, 64, channels, r, ldy=ld, flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0, **kw)
        Gr = torch.full((channels, r) if w_oi else (r, channels), 7.0, device=dev).bfloat16()
        dX = torch.empty(n, 64, device=dev, dtype=torch.bfloat16)
        acc.acc_linear_bwd(bdesc, X, W if w_oi else W.T.contiguous(), None, dX, Gr, None, acc.alloc_workspace(bdesc, True, dev))
        got.append(Gr if w_oi else Gr.T)
    want = X.double().T @ S.double()
    bound = want.abs() * 2.0 ** -8 + 12 * 4 * 2.0 ** -24 * 4096 ** 0.5 * want.square().mean().sqrt()
    for v in got:
        over = float(((v.double() - want).abs() / bound).max())
        assert over <= 1.0, over
