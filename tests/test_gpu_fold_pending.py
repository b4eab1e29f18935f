"""The sketch's partial tiles folded by the launch of the exact product behind it, for every count of splits that the groups of eight
reads leave over, on the ring kernel, the persistent one and the 8-bit one: against a product in 64 bits with the device's own S.

Bound: the factor is float and its operands are exact in bfloat16, so only the fp32 sums round: 256 tokens in a split and the splits'
sum, 4 2^-24 sqrt(256 + splits) of the root mean square; 12 times that for the largest of many entries.  A split left out or added twice
is off by 1 / sqrt(splits)."""
import pytest

import plan_util as plan

pytestmark = pytest.mark.gpu

CHANNELS, RANK = 640, 72


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


@pytest.mark.parametrize("splits,persistent", [(2, 25600), (3, 17408), (4, 13312), (5, 11264), (6, 9216), (7, 8192), (8, 7168), (9, 6144),
                                               (10, 6144), (12, 5120), (16, 4096), (17, 3072), (18, 3072)])
def test_fold(acc, splits, persistent):
    import torch
    dev, n = "cuda:0", 256 * splits - 24
    p = plan.sketch(n, CHANNELS, RANK, bf16_factor=False)
    assert p.tuned and p.splits == splits and p.tokens == 256
    assert plan.gemm_tile(n, 64, CHANNELS)[0] == "64x64" and plan.gemm_tile(n, persistent, CHANNELS)[0] == "256x256"
    g = torch.Generator(device=dev).manual_seed(splits)
    X = torch.randn(n, CHANNELS, generator=g, device=dev).bfloat16()
    kw = dict(seed=5, row_offset=12, factor_dtype=acc.ACC_F32)
    S = torch.empty(n, RANK, device=dev)
    got = {}
    for kernel, d_out in (("ring", 64), ("persistent", persistent), ("8-bit", 512)):
        desc = acc.make_desc(n, CHANNELS, d_out, RANK, **kw)
        Y, Xs = torch.empty(n, d_out, device=dev, dtype=torch.bfloat16), torch.full((CHANNELS, RANK), 7.0, device=dev)
        ws = acc.alloc_workspace(desc, False, dev)
        print(f"fold {splits} splits, {kernel}", flush=True)
        if kernel == "8-bit":
            X8, W8 = (torch.zeros(s, dtype=torch.uint8, device=dev) for s in ((n, CHANNELS), (CHANNELS, d_out)))
            acc.acc_linear_fwd_fp8(desc, X, X8, W8, 1.0, Y, Xs, ws)
        else:
            acc.acc_linear_fwd(desc, X, torch.zeros(CHANNELS, d_out, device=dev, dtype=torch.bfloat16), Y, Xs, ws)
        got[kernel] = Xs
    acc.acc_sketch_dump(desc, S)
    want = X.double().T @ S.double()
    rms, tol = want.square().mean().sqrt(), 4 * 2.0 ** -24 * (256 + splits) ** 0.5
    for kernel, v in got.items():
        over = (v.double() - want).abs() / rms
        assert float(over.square().mean().sqrt()) <= tol and float(over.max()) <= 12 * tol, kernel
        assert torch.equal(v, got["ring"]), kernel   # one order of the sums
