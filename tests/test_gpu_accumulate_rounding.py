"""A product that is added to a bfloat16 result is rounded once: the sum, not the product and then the sum.  Dense gradients
accumulated in every kernel of the factors' product, and the optimizer's update of the weight, at ranks that are and that are
no multiple of 64.

Bound per element: half a unit in the last place of the exact sum in bfloat16, plus the float32 sum's own rounding,
2^-24 (sqrt(r) + 3) of the largest that the terms' absolute values can add up to."""
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


def _rounded_once(got, want, size, r):
    import torch
    half = torch.exp2(torch.floor(torch.log2(want.abs().clamp_min(1e-30))) - 8)
    excess = ((got.double() - want).abs() - half - 2.0 ** -24 * (r ** 0.5 + 3) * size).max()
    assert excess <= 0, float(excess / half.median())


@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("d_in,d_out,r,tile", [
    (200, 392, 32, "64x64"),             # half a K tile
    (1000, 1160, 64, "64x64"),
    (520, 1032, 1096, "64x64"),
    (3264, 3080, 40, "128x64"),
    (4104, 3080, 32, "128x64"),
    (4104, 3080, 128, "128x64"),
    (3064, 2968, 40, "three-stage"),     # one K tile, masked
    (2968, 3064, 264, "three-stage"),    # five, the last one masked
    (8200, 8200, 64, "three-stage"),     # more tiles than compute units
    (8200, 6152, 200, "192x128"),
])
def test_accumulated_gradient(acc, d_in, d_out, r, tile, w_oi):
    import torch
    assert plan.factor_tile(*((d_out, d_in) if w_oi else (d_in, d_out)), r, added=True) == tile
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(d_in + r)
    left = torch.randn(d_in, r, generator=g, device=dev).bfloat16()
    Gr = torch.randn(r, d_out, generator=g, device=dev).bfloat16()
    before = (torch.randn(d_in, d_out, generator=g, device=dev) * r ** 0.5).bfloat16()
    T = (lambda a: a.T.contiguous()) if w_oi else (lambda a: a.clone())
    dW = T(before)
    desc = acc.make_desc(1, d_in, d_out, r, io_dtype=acc.ACC_BF16,
                         flags=acc.ACC_FLAG_DW_ACCUMULATE | (acc.ACC_FLAG_W_OUT_IN if w_oi else 0))
    print(f"accumulate {d_in} x {d_out} r={r} w_oi={w_oi}", flush=True)
    acc.acc_linear_dw(desc, left, T(Gr), dW)
    want = T(before.double() + left.double() @ Gr.double())
    size = T(before.double().abs() + left.double().abs() @ Gr.double().abs())
    _rounded_once(dW, want, size, r)


@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("d_in,d_out,r", [(520, 264, 8), (520, 264, 32), (1032, 1544, 64), (3264, 3080, 96)])
def test_weight_update(acc, d_in, d_out, r, w_oi):
    """With both betas and eps zero the normalised step is the sign of the small factor, so the update is known exactly."""
    import numpy as np
    import torch
    dev = "cuda:0"
    g = torch.Generator(device=dev).manual_seed(d_in + r)
    left = torch.randn(d_in, r, generator=g, device=dev).bfloat16()
    Gr = (torch.rand(r, d_out, generator=g, device=dev) + 0.5).bfloat16()
    Gr *= torch.randint(0, 2, (r, d_out), generator=g, device=dev).bfloat16() * 2 - 1
    W = torch.randn(d_in, d_out, generator=g, device=dev).bfloat16()
    T = (lambda a: a.T.contiguous()) if w_oi else (lambda a: a.clone())
    Wg, M, V = T(W), T(torch.zeros(r, d_out, device=dev)), T(torch.zeros(r, d_out, device=dev))
    desc = acc.make_desc(1, d_in, d_out, r, io_dtype=acc.ACC_BF16, flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0)
    hyper = acc.make_hyper(step=1, lr=0.25, beta1=0.0, beta2=0.0, eps=0.0, weight_decay=0.5, scale=0.75)
    print(f"weight update {d_in} x {d_out} r={r} w_oi={w_oi}", flush=True)
    acc.acc_lowrank_adamw_step(desc, hyper, None, 0, left, T(Gr), M, V, Wg, acc.alloc_lowrank_workspace(desc, 0, dev))
    beta = float(np.float32(1) - np.float32(0.25) * np.float32(0.5))
    step = 0.25 * 0.75 * (left.double() @ torch.sign(Gr).double())
    want = T(beta * W.double() - step)
    size = T(W.double().abs() + 0.25 * 0.75 * left.double().abs().sum(1, keepdim=True))
    _rounded_once(Wg, want, size, r)
