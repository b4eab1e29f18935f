"""The bfloat16 sketch with bfloat16 factors, whose slabs and token splits pick_sketch_split chooses: one running sum and two (of even
and odd 32-token stages), ragged last slab, ragged last split, an odd and an even number of stages, surplus sketch columns, padded
rows, both orientations, against a product in 64 bits with the device's own S.

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


def _factors(acc, n, channels, r, X):
    """Xs, and Gr of a backward pass with `channels` outputs in both orientations: the same product three times, [channels, r]."""
    import torch
    dev = "cuda:0"
    W = torch.zeros(channels, 64, device=dev).bfloat16()   # the products are not looked at here
    kw = dict(seed=11, row_offset=40)
    desc = acc.make_desc(n, channels, 64, r, ldx=X.stride(0), **kw)
    S = torch.empty(n, r, device=dev)
    acc.acc_sketch_dump(desc, S)
    Y, Xs = torch.empty(n, 64, device=dev, dtype=torch.bfloat16), torch.full((channels, r), 7.0, device=dev).bfloat16()
    acc.acc_linear_fwd(desc, X, W, Y, Xs, acc.alloc_workspace(desc, False, dev))
    got = [Xs]
    for w_oi in (False, True):
        bdesc = acc.make_desc(n, 64, channels, r, ldy=X.stride(0), flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0, **kw)
        Gr = torch.full((channels, r) if w_oi else (r, channels), 7.0, device=dev).bfloat16()
        dX = torch.empty(n, 64, device=dev, dtype=torch.bfloat16)
        acc.acc_linear_bwd(bdesc, X, W if w_oi else W.T.contiguous(), None, dX, Gr, None, acc.alloc_workspace(bdesc, True, dev))
        got.append(Gr if w_oi else Gr.T)
    return S, got


@pytest.mark.parametrize("n,channels,r,pad,slab,two_sums", [
    (300, 3064, 256, 0, 128, False), (601, 2056, 200, 8, 128, False), (1030, 520, 72, 0, 128, False), (31, 264, 24, 0, 128, False),
    (4097, 8184, 256, 8, 512, False), (8190, 3080, 200, 8, 512, False),
    (4095, 4088, 128, 0, 256, True), (2050, 4096, 232, 16, 256, True), (8190, 2056, 128, 0, 256, True), (700, 3064, 512, 8, 256, True),
    (4090, 1016, 248, 0, 128, True),
])
def test_sketch(acc, n, channels, r, pad, slab, two_sums):
    import torch
    p = plan.sketch(n, channels, r, ld=channels + pad)
    assert (p.slab, p.two_sums) == (slab, two_sums)
    g = torch.Generator(device="cuda:0").manual_seed(n + r)
    X = torch.randn(n, channels + pad, generator=g, device="cuda:0").bfloat16()[:, :channels]
    print(f"sketch {n} x {channels} rank {r}", flush=True)
    S, got = _factors(acc, n, channels, r, X)
    want = X.double().T @ S.double()
    bound = want.abs() * 2.0 ** -8 + 12 * 4 * 2.0 ** -24 * 4096 ** 0.5 * want.square().mean().sqrt()
    for v in got:
        over = float(((v.double() - want).abs() / bound).max())
        assert over <= 1.0, over


def far_apart(S, tokens, n, channels):
    """X [n, channels] whose sums with S are lost in a running sum of all of a split's tokens and kept in one of even and one of odd
    stages.  For channel c and sketch column c mod r, in the first split: one large product in stage 0, taken back by the last three
    even stages (each takes what the bfloat16 entries before it leave, 2^-9 of it), and small ones of 2^-26 in the odd stages
    before those, which add up to the result."""
    import torch
    dev, r = S.device, S.shape[1]
    cols = torch.arange(channels, device=dev) % r
    X = torch.zeros(n, channels, device=dev, dtype=torch.float64)
    at = torch.arange(channels, device=dev)

    def place(first, count, product):   # the token of [first, first + count) with the largest entry of S takes `product`
        t = S[first:first + count, cols].abs().argmax(0) + first
        s = S[t, cols].double()
        x = (product / s).bfloat16().double()
        X[t, at] = x
        return x * s
    left = place(0, 32, torch.ones(channels, device=dev, dtype=torch.float64))
    large = left.clone()
    last = (min(tokens, n) // 32 - 1) // 2 * 2
    for stage in (last - 4, last - 2, last):
        left = left + place(32 * stage, 32, -left)
    for stage in range(1, last - 4, 2):
        for half in (0, 16):
            place(32 * stage + half, 16, large * 2.0 ** -26)
    return X.bfloat16(), cols


@pytest.mark.parametrize("n,channels,r,slab", [(2050, 4096, 232, 256), (8190, 2056, 128, 256), (4090, 1016, 248, 128)])
def test_small_terms_outlive_a_large_one_of_the_other_stages(acc, n, channels, r, slab):
    """Fewer splits of more tokens do not make running sums longer: the sums of even and of odd stages are apart.  Apart, both
    are exact to a few units of 2^-24 and the result rounds once to bfloat16, 2^-9.  In one running sum every small term is at most half
    of half a unit in the last place of the large one, and all of them are gone."""
    import torch
    p = plan.sketch(n, channels, r)
    assert p.two_sums and p.slab == slab
    desc = acc.make_desc(n, channels, 64, r, seed=11, row_offset=40)
    S = torch.empty(n, r, device="cuda:0")
    acc.acc_sketch_dump(desc, S)
    X, cols = far_apart(S, p.tokens, n, channels)
    print(f"sketch sums {n} x {channels} rank {r}", flush=True)
    S, got = _factors(acc, n, channels, r, X)
    rows = torch.arange(channels, device="cuda:0")
    want = (X.double() * S.double()[:, cols]).sum(0)
    for v in got:
        err = (v[rows, cols].double() - want).abs() / want.abs()
        assert float(err.max()) <= 2.0 ** -7, (float(err.max()), float(err.mean()))
