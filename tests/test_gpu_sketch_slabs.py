"""The bfloat16 sketch on slabs of 128, 256 and 512 channels: ragged last slab, ragged last token stage, surplus sketch columns, padded
rows, both orientations, against a product in 64 bits with the device's own S.

Bound: S and the input are exact in bfloat16 and the factor is float, so only the fp32 sums round: the tokens of a split's
running sum and the splits' sum, 4 2^-24 sqrt(tokens + splits) of the root mean square; 12 times that for the largest of many entries."""
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
    (300, 136, 8, 0, 128), (257, 128, 64, 0, 128), (31, 264, 24, 8, 128), (2049, 1032, 128, 0, 128), (1030, 2040, 72, 24, 128),
    (4096, 1024, 256, 0, 256), (1001, 3976, 200, 16, 256), (2500, 1544, 152, 0, 256),
    (2500, 2056, 152, 0, 512), (2048, 2040, 512, 0, 512), (8190, 3080, 200, 8, 512),
])
def test_sketch(acc, n, channels, r, pad, slab):
    import torch
    p = plan.sketch(n, channels, r, bf16_factor=False, ld=channels + pad)
    assert p.slab == slab and not p.two_sums
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(n + r)
    ld = channels + pad
    X = torch.randn(n, ld, generator=g, device=dev).bfloat16()[:, :channels]
    W = torch.randn(channels, 64, generator=g, device=dev).bfloat16()
    kw = dict(seed=11, row_offset=40, factor_dtype=acc.ACC_F32)
    desc = acc.make_desc(n, channels, 64, r, ldx=ld, **kw)
    S = torch.empty(n, r, device=dev)
    acc.acc_sketch_dump(desc, S)
    Y, Xs = torch.empty(n, 64, device=dev, dtype=torch.bfloat16), torch.full((channels, r), 7.0, device=dev)
    print(f"sketch {n} x {channels} rank {r}", flush=True)
    acc.acc_linear_fwd(desc, X, W, Y, Xs, acc.alloc_workspace(desc, False, dev))
    got = [Xs]
    for w_oi in (False, True):   # the small factor of a backward pass with `channels` outputs is the same product
        bdesc = acc.make_desc(n, 64, channels, r, ldy=ld, flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0, **kw)
        Gr = torch.full((channels, r) if w_oi else (r, channels), 7.0, device=dev)
        dX = torch.empty(n, 64, device=dev, dtype=torch.bfloat16)
        acc.acc_linear_bwd(bdesc, X, W if w_oi else W.T.contiguous(), None, dX, Gr, None, acc.alloc_workspace(bdesc, True, dev))
        got.append(Gr if w_oi else Gr.T)
    want = X.double().T @ S.double()
    rms = want.square().mean().sqrt()
    tol = 4 * 2.0 ** -24 * (p.tokens + p.splits) ** 0.5
    for v in got:
        err, worst = float((v.double() - want).square().mean().sqrt() / rms), float((v.double() - want).abs().max() / rms)
        assert err <= tol and worst <= 12 * tol, (err, worst)
