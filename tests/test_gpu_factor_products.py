"""The optimizer's products of bfloat16 and float32 factors on the float32 kernel, at sizes that take its 64 x 64 and its
32 x 32 tiles, with ranks that end inside a tile and inside a K tile.

Bounds: the moments come from products of exact operands summed in fp32 (r + d_in terms: 2^-24 sqrt of that, times four)
and from 1 - beta formed in fp32 (1 - 0.999f is off by 2e-5 of itself at most, seen only in V); the weight rounds the step
and the sum once each."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import acc_oracle as orc
import gpu_util as gu


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


@pytest.mark.parametrize("w_oi", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_in,d_out,r,k", [(72, 40, 24, 8), (1032, 520, 72, 40), (8184, 8184, 264, 256)])
def test_step_and_projector(acc, d_in, d_out, r, k, dtype, w_oi):
    import torch
    dev = "cuda:0"
    t, code = (torch.float32, acc.ACC_F32) if dtype == "f32" else (torch.bfloat16, acc.ACC_BF16)
    g = torch.Generator(device=dev).manual_seed(d_in + r)
    randn = lambda *s: torch.randn(*s, generator=g, device=dev)  # noqa: E731
    left, Gr, W = randn(d_in, r).to(t), (randn(r, d_out) * 0.01).to(t), (randn(d_in, d_out) * 0.02).to(t)
    P = torch.linalg.qr(randn(d_in, k).cpu())[0].contiguous().to(dev).to(t)
    M, V = randn(k, d_out) * 0.1, torch.rand(k, d_out, generator=g, device=dev) * 0.01
    h = dict(step=3, lr=0.05, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.1, scale=1.0)
    T = (lambda a: a.T.contiguous()) if w_oi else (lambda a: a.clone())
    Wg, Mg, Vg, Grg, Pr = T(W), T(M), T(V), T(Gr), torch.full((d_in, k), 7.0, dtype=t, device=dev)
    desc = acc.make_desc(1, d_in, d_out, r, seed=9, io_dtype=code, flags=acc.ACC_FLAG_W_OUT_IN if w_oi else 0)
    ws = acc.alloc_lowrank_workspace(desc, k, dev)
    print(f"step and projector {d_in} x {d_out} r={r} k={k} {dtype} w_oi={w_oi}", flush=True)
    acc.acc_lowrank_adamw_step(desc, acc.make_hyper(**h), P, k, left, Grg, Mg, Vg, Wg, ws)
    acc.acc_lowrank_projector(desc, k, left, Grg, Pr, ws)
    torch.cuda.synchronize()
    U = (lambda a: a.T.double()) if w_oi else (lambda a: a.double())
    R = (P.double().T @ left.double()) @ Gr.double()
    Mw = h["beta1"] * M.double() + (1 - h["beta1"]) * R
    Vw = h["beta2"] * V.double() + (1 - h["beta2"]) * R * R
    N = (Mw / (1 - h["beta1"] ** 3)) / (torch.sqrt(Vw / (1 - h["beta2"] ** 3)) + h["eps"])
    Ww = (1 - h["lr"] * h["weight_decay"]) * W.double() - h["lr"] * (P.double() @ N)
    rel = lambda a, b: float((a - b).norm() / b.norm())  # noqa: E731
    e = 4 * 2.0 ** -24 * (r + d_in) ** 0.5 + 1e-6
    errs = {"M": rel(U(Mg), Mw), "V": rel(U(Vg), Vw), "W": rel(U(Wg), Ww)}
    print("  ", errs, flush=True)
    assert errs["M"] <= e and errs["V"] <= e + 2e-5
    # a bfloat16 weight rounds N (an operand), the step and the sum
    assert errs["W"] <= (e + 2e-5 if dtype == "f32" else 3 * 2.0 ** -9)
    omega = torch.from_numpy(orc.range_finder_matrix(9, d_out, k)).to(dev)
    Yp = left.double() @ (Gr.double() @ omega)
    q, upper = np.linalg.qr(Yp.cpu().numpy())
    want = q * np.sign(np.diag(upper))
    cond = np.linalg.cond(Yp.cpu().numpy())
    err = gu.rel(acc.to_host_f64(Pr), want)
    print(f"   P {err:.2e} cond {cond:.0f}", flush=True)
    assert err <= cond * 1e-6 + (0 if dtype == "f32" else 2.0 ** -9)
