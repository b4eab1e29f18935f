"""The work that a user of the compressed linear layer has it do, as measurable cases.

A case is one pass through the public entry points (`binding`, `autograd`): a layer's forward and backward, the
optimizer step on the gradient factors, or the refresh of its projector.  `listed()` names the fixed cases, `draw()`
gives more of the same ranges, `prepare()` makes what a program holds before the call, `run()` is the call and
`exact()` its result in 64 bits.

kind        what one pass is
  layer     acc_linear_fwd + acc_linear_bwd with the dense dW, outputs and workspaces kept by the caller
  module    the autograd function in torch.nn.Linear's weight layout: y, then the gradients of x, weight and bias
  qkv       three linears on one input (the sketch taken once), forward and backward
  rsvd      acc_linear_fwd_rsvd + acc_linear_bwd_rsvd with the dense dW
  fp8       the layer with its exact products on 8-bit operands
  adamw     one acc_lowrank_adamw_step through a projector
  refresh   one acc_lowrank_projector
"""
import math

import torch

from paper_2605_01255_amd import binding as acc
from paper_2605_01255_amd.autograd import CompressedLinearFunction

DEV = "cuda:0"
ADAM = {"step": 10, "lr": 1e-3, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8, "weight_decay": 0.01, "scale": 1.0}


def listed():
    return [
        # the tiny fp32 layer of the repository's first configuration: launches and their latency are all there is
        {"name": "tiny_f32", "kind": "layer", "n": 256, "d_in": 256, "d_out": 512, "r": 16, "dtype": "f32"},
        # a short batch (a few hundred tokens) through a 3B-shaped projection with bias, as a fine-tuning loop calls it
        {"name": "short_batch_bias", "kind": "module", "n": 384, "d_in": 3072, "d_out": 3072, "r": 64, "dtype": "bf16",
         "bias": True, "compressor": "rp", "power": 0},
        # sizes that are no multiples of a tile: an odd number of tokens, odd widths
        {"name": "ragged_bf16", "kind": "layer", "n": 2049, "d_in": 1032, "d_out": 1544, "r": 128, "dtype": "bf16"},
        # a float32 layer of ordinary size with bias
        {"name": "f32_bias", "kind": "module", "n": 2048, "d_in": 1024, "d_out": 2048, "r": 64, "dtype": "f32", "bias": True,
         "compressor": "rp", "power": 0},
        # the attention inputs of a 3B-shaped decoder layer on one sequence: q, k and v share their input's sketch
        {"name": "qkv_sequence", "kind": "qkv", "n": 4096, "d_in": 3072, "d_out": 3072, "d_kv": 1024, "r": 256,
         "dtype": "bf16"},
        # the headline workload: 3B-shaped attention projection, forward, backward and dense dW
        {"name": "attn_proj", "kind": "layer", "n": 16384, "d_in": 3072, "d_out": 3072, "r": 256, "dtype": "bf16"},
        # the same on 8-bit operands
        {"name": "attn_proj_fp8", "kind": "fp8", "n": 16384, "d_in": 3072, "d_out": 3072, "r": 256, "dtype": "bf16"},
        # the largest: down projection of an 8B-shaped MLP on 65536 tokens
        {"name": "mlp_down_8b", "kind": "module", "n": 65536, "d_in": 14336, "d_out": 4096, "r": 512, "dtype": "bf16",
         "bias": False, "compressor": "rp", "power": 0},
        # the more accurate compressor at the paper's rank
        {"name": "rsvd_rank32", "kind": "rsvd", "n": 16384, "d_in": 3072, "d_out": 3072, "r": 32, "dtype": "bf16", "power": 0},
        # and at a rank that needs the blocked factorisation, with a round of subspace iteration
        {"name": "rsvd_rank128_power", "kind": "module", "n": 4096, "d_in": 2048, "d_out": 2048, "r": 128, "dtype": "bf16",
         "bias": False, "compressor": "rsvd", "power": 1},
        # the optimizer's update of a 3B-shaped projection from its gradient factors
        {"name": "adamw_step", "kind": "adamw", "d_in": 3072, "d_out": 3072, "r": 256, "k": 64, "dtype": "bf16"},
        # the refresh of the optimizer's projector
        {"name": "projector_refresh", "kind": "refresh", "d_in": 3072, "d_out": 3072, "r": 256, "k": 128, "dtype": "bf16"},
    ]


LARGEST = 65536 * 14336 * 4096   # multiply-adds of one exact product of the largest listed case


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi):
    """A layer width: most are multiples of 64 as in trained models, one in four only of 8."""
    q = 8 if rng.random() < 0.25 else 64
    return max(lo // q * q or q, int(_log(rng, lo, hi)) // q * q)


def draw(rng):
    kind = rng.choice(["layer", "layer", "module", "module", "qkv", "rsvd", "fp8", "adamw", "refresh"])
    f32 = kind not in ("fp8", "qkv") and rng.random() < 0.25
    top = 4096 if f32 else 14336
    rank = [16, 32, 64, 128, 256] if f32 else [8, 16, 24, 32, 64, 128, 256, 512]
    while True:
        c = {"kind": kind}
        if kind in ("adamw", "refresh"):
            c["d_in"], c["d_out"] = _width(rng, 512, min(top, 8192)), _width(rng, 512, min(top, 8192))
            c["r"] = rng.choice([64, 128, 256, 512])
            c["k"] = rng.choice([k for k in (8, 16, 32, 64, 96, 128, 256) if k <= c["r"]])
            c["dtype"] = "f32" if f32 else "bf16"
            return c
        c["n"] = int(_log(rng, 256, 4096 if f32 else 65536))
        c["d_in"], c["d_out"] = _width(rng, 256, top), _width(rng, 256, top)
        c["r"] = rng.choice(rank)
        c["dtype"] = "f32" if f32 else "bf16"
        if kind == "module":
            c["bias"] = rng.random() < 0.5
            c["compressor"] = rng.choice(["rp", "rp", "rp", "rsvd"])
            c["power"] = rng.choice([0, 1]) if c["compressor"] == "rsvd" else 0
        if kind == "rsvd":
            c["power"] = rng.choice([0, 0, 1])
        if kind == "qkv":
            c["d_kv"] = max(256, c["d_out"] // rng.choice([1, 2, 4, 8]) // 8 * 8)
        if kind == "fp8":
            c["d_in"], c["d_out"] = max(512, c["d_in"] // 128 * 128), max(512, c["d_out"] // 128 * 128)
        if kind == "rsvd" or c.get("compressor") == "rsvd":
            c["r"] = min(c["r"], 256)
            if c["r"] * 4 > min(c["n"], c["d_in"]):
                continue
        ragged = c["d_in"] % 64 or c["d_out"] % 64
        if c["n"] * c["d_in"] * c["d_out"] <= LARGEST // (128 if f32 else 32 if ragged else 4):
            return c


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, rows, cols, scale, dtype):
    return (torch.randn(rows, cols, generator=g, device=DEV) * scale).to(dtype)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _code(case):
    return acc.ACC_F32 if case["dtype"] == "f32" else acc.ACC_BF16


def _activations(g, n, d, dtype):
    """Token rows ~ N(0, 1) with eight feature channels of twenty times the size, as activations of a language model."""
    x = torch.randn(n, d, generator=g, device=DEV)
    x[:, [j * (d // 8) + 5 for j in range(8)]] *= 20.0
    return x.to(dtype)


def _tensors(case, seed):
    """The inputs alone, from the seed."""
    g, t = _gen(seed), _dtype(case)
    kind = case["kind"]
    d_in, d_out, r = case["d_in"], case["d_out"], case["r"]
    if kind in ("adamw", "refresh"):
        s = math.sqrt(16384 / r)
        out = {"left": _randn(g, d_in, r, s, t), "Gr": _randn(g, d_out, r, 0.01 * s, t)}
        if kind == "adamw":   # the [out, in] layout; moments as nine earlier steps leave them
            k = case["k"]
            out["P"] = torch.linalg.qr(torch.randn(d_in, k, generator=g, device=DEV).cpu())[0].contiguous().to(DEV).to(t)
            size = 0.01 * s * s * math.sqrt(r)
            out["M"] = torch.randn(d_out, k, generator=g, device=DEV) * (0.3 * size)
            out["V"] = torch.rand(d_out, k, generator=g, device=DEV) * (0.01 * size * size)
            out["W"] = _randn(g, d_out, d_in, 0.02, t)
        return out
    out = {"X": _activations(g, case["n"], d_in, t)}
    if kind == "qkv":
        widths = (d_out, case["d_kv"], case["d_kv"])
        out["W"] = [_randn(g, d_in, w, 0.02, t) for w in widths]
        out["dY"] = [_randn(g, case["n"], w, 0.01, t) for w in widths]
        return out
    shape = (d_out, d_in) if kind == "module" else (d_in, d_out)
    out["W"] = _randn(g, *shape, 0.02, t)
    out["dY"] = _randn(g, case["n"], d_out, 0.01, t)
    if case.get("bias"):
        out["b"] = (torch.randn(d_out, generator=g, device=DEV) * 0.1).to(t)
    if kind == "fp8":
        for name in ("X", "W", "dY"):
            scale = 2.0 ** math.ceil(math.log2(float(out[name].abs().max()) / 448.0))
            out[name + "8"] = (out[name].float() / scale).to(torch.float8_e4m3fn).view(torch.uint8)
            out[name + "_scale"] = scale
    return out


def _empty(t, *shape):
    return torch.empty(*shape, dtype=t, device=DEV)


def prepare(case, seed):
    s = {"case": case, "seed": seed, **_tensors(case, seed)}
    t, code, kind = _dtype(case), _code(case), case["kind"]
    d_in, d_out, r = case["d_in"], case["d_out"], case["r"]
    if kind in ("adamw", "refresh"):
        k = case["k"]
        s["desc"] = acc.make_desc(1, d_in, d_out, r, seed=seed, io_dtype=code, flags=acc.ACC_FLAG_W_OUT_IN)
        s["ws"] = acc.alloc_lowrank_workspace(s["desc"], k, DEV)
        if kind == "adamw":
            s["hyper"] = acc.make_hyper(**ADAM)
        else:
            s["P"] = _empty(t, d_in, k)
        return s
    n = case["n"]
    if kind == "module":
        s["X"].requires_grad_(True)
        s["W"].requires_grad_(True)
        if case["bias"]:
            s["b"].requires_grad_(True)
        return s
    if kind == "qkv":
        parts = []
        for i, (W, dY) in enumerate(zip(s["W"], s["dY"])):
            w = W.shape[1]
            parts.append({"fd": acc.make_desc(n, d_in, w, r, seed=seed, io_dtype=code,
                                              flags=acc.ACC_FLAG_SKIP_SKETCH if i else 0),
                          "bd": acc.make_desc(n, d_in, w, r, seed=seed, io_dtype=code),
                          "Y": _empty(t, n, w), "dX": _empty(t, n, d_in), "Gr": _empty(t, r, w), "dW": _empty(t, d_in, w)})
        s["parts"], s["Xs"] = parts, _empty(t, d_in, r)
        s["ws_f"] = acc.alloc_workspace(parts[0]["bd"], False, DEV)
        s["ws_b"] = acc.alloc_workspace(max((p["bd"] for p in parts), key=lambda d: acc.acc_linear_workspace_bytes(d, True)),
                                        True, DEV)
        return s
    rsvd = kind == "rsvd"
    s["desc"] = acc.make_desc(n, d_in, d_out, r, seed=seed, io_dtype=code,
                              flags=case.get("power", 0) << acc.ACC_FLAG_RSVD_POWER_SHIFT if rsvd else 0)
    s["ws_f"] = acc.alloc_workspace(s["desc"], False, DEV, rsvd=rsvd)
    s["ws_b"] = acc.alloc_workspace(s["desc"], True, DEV, rsvd=rsvd)
    s["Y"], s["dX"], s["Gr"], s["dW"] = _empty(t, n, d_out), _empty(t, n, d_in), _empty(t, r, d_out), _empty(t, d_in, d_out)
    s["Xs"] = _empty(t, d_in, r)
    if rsvd:
        s["U"] = _empty(t, n, r)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "layer":
        acc.acc_linear_fwd(s["desc"], s["X"], s["W"], s["Y"], s["Xs"], s["ws_f"])
        acc.acc_linear_bwd(s["desc"], s["dY"], s["W"], s["Xs"], s["dX"], s["Gr"], s["dW"], s["ws_b"])
        return {k: s[k] for k in ("Y", "Xs", "dX", "Gr", "dW")}
    if kind == "module":
        b = s.get("b")
        y = CompressedLinearFunction.apply(s["X"], s["W"], b, case["r"], s["seed"], case["compressor"], case["power"], None)
        wrt = (s["X"], s["W"]) if b is None else (s["X"], s["W"], b)
        grads = torch.autograd.grad(y, wrt, s["dY"])
        return dict(zip(("Y", "dX", "dW", "dB"), (y.detach(), *grads)))
    if kind == "qkv":
        for i, (p, W) in enumerate(zip(s["parts"], s["W"])):
            acc.acc_linear_fwd(p["fd"], s["X"], W, p["Y"], s["Xs"], None if i else s["ws_f"])
        for p, W, dY in zip(reversed(s["parts"]), reversed(s["W"]), reversed(s["dY"])):
            acc.acc_linear_bwd(p["bd"], dY, W, s["Xs"], p["dX"], p["Gr"], p["dW"], s["ws_b"])
        return [s["Xs"], [{k: p[k] for k in ("Y", "dX", "Gr", "dW")} for p in s["parts"]]]
    if kind == "rsvd":
        acc.acc_linear_fwd_rsvd(s["desc"], s["X"], s["W"], s["Y"], s["U"], s["Xs"], s["ws_f"])
        acc.acc_linear_bwd_rsvd(s["desc"], s["dY"], s["W"], s["U"], s["Xs"], s["dX"], s["Gr"], s["dW"], s["ws_b"])
        return {"Y": s["Y"], "U": s["U"], "V": s["Xs"], "dX": s["dX"], "Gr": s["Gr"], "dW": s["dW"]}
    if kind == "fp8":
        acc.acc_linear_fwd_fp8(s["desc"], s["X"], s["X8"], s["W8"], s["X_scale"] * s["W_scale"], s["Y"], s["Xs"], s["ws_f"])
        acc.acc_linear_bwd_fp8(s["desc"], s["dY"], s["dY8"], acc.ACC_FP8_E4M3, s["W8"], s["dY_scale"] * s["W_scale"], s["Xs"],
                               s["dX"], s["Gr"], s["dW"], s["ws_b"])
        return {k: s[k] for k in ("Y", "Xs", "dX", "Gr", "dW")}
    if kind == "adamw":
        acc.acc_lowrank_adamw_step(s["desc"], s["hyper"], s["P"], case["k"], s["left"], s["Gr"], s["M"], s["V"], s["W"], s["ws"])
        return {"M": s["M"], "V": s["V"], "W": s["W"]}
    acc.acc_lowrank_projector(s["desc"], case["k"], s["left"], s["Gr"], s["P"], s["ws"])
    return {"P": s["P"]}


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def work(case):
    kind, e = case["kind"], 4 if case["dtype"] == "f32" else 2
    d_in, d_out, r = case["d_in"], case["d_out"], case["r"]
    if kind == "adamw":
        k = case["k"]
        return {"bytes": e * (d_in * (k + r) + r * d_out + 2 * d_in * d_out) + 16 * k * d_out,
                "flops": 2 * (k * d_in * r + k * r * d_out + d_in * k * d_out)}
    if kind == "refresh":
        k = case["k"]
        return {"bytes": e * (d_in * (r + k) + r * d_out), "flops": 2 * (r * d_out * k + d_in * r * k + 2 * d_in * k * k)}
    n = case["n"]
    if kind == "qkv":
        w = d_out + 2 * case["d_kv"]
        return {"bytes": e * (n * d_in + d_in * r + 2 * (d_in * w + n * w) + 3 * n * d_in + r * w),
                "flops": 4 * n * d_in * w + 2 * n * r * (d_in + w) + 2 * d_in * r * w}
    flops = 4 * n * d_in * d_out + 2 * n * r * (d_in + d_out) + 2 * d_in * r * d_out
    size = e * (2 * n * (d_in + d_out) + 2 * d_in * d_out + r * (d_in + d_out))
    if kind == "fp8":
        size += n * (d_in + d_out) - d_in * d_out
    if kind == "rsvd" or case.get("compressor") == "rsvd":
        flops += 2 * n * d_in * r * (1 + 2 * case["power"]) + 4 * n * r * r
        size += e * n * r
    return {"bytes": size, "flops": flops}


def tolerance(case):
    if case["dtype"] == "f32":
        # sums of a few thousand terms in 32 bits; the moments' 1 - beta2 is formed in 32 bits; an orthonormal factor
        # carries the condition of what it factors, worst where the projector's rank reaches the gradient's
        if case["kind"] == "refresh":
            return {"rel": 7e-5}
        if case["kind"] == "adamw":
            return {"rel": 1.5e-5}
        return {"rel": 1e-5 if case["kind"] == "rsvd" or case.get("compressor") == "rsvd" else 5e-6}
    return {"rel": 1e-2}


# ---- the results in 64 bits ------------------------------------------------------------------------------------------
def _normals(seed, count, cols):
    """S [count, cols]: Philox4x32-10 with counter (row >> 2, column), four rows a call, Box-Muller, over sqrt(cols)."""
    mask = 0xFFFFFFFF
    q = torch.arange((count + 3) // 4, device=DEV)[:, None]
    c = [q & mask, torch.arange(cols, device=DEV)[None, :], torch.zeros_like(q), q >> 32]
    k = [seed & mask, seed >> 32 & mask]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # the low 64 bits, whatever the sign
        c = [p1 >> 32 & mask ^ c[1] ^ k[0], p1 & mask, p0 >> 32 & mask ^ c[3] ^ k[1], p0 & mask]
        k = [(k[0] + 0x9E3779B9) & mask, (k[1] + 0xBB67AE85) & mask]
    u = [((x >> 9).double() + 0.5) * 2.0 ** -23 for x in torch.broadcast_tensors(*c)]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        radius, angle = torch.sqrt(-2.0 * torch.log(a)), 2.0 * math.pi * b
        z += [radius * torch.cos(angle), radius * torch.sin(angle)]
    return torch.stack(z, 1).reshape(-1, cols)[:count] / math.sqrt(cols)


def _orth(y):
    """Thin QR factor with a positive diagonal of R (Cholesky twice and once more, in 64 bits)."""
    for _ in range(3):
        upper = torch.linalg.cholesky((y.T @ y).cpu()).T
        y = y @ torch.linalg.inv(upper).to(DEV)
    return y


def exact(case, seed):
    s = _tensors(case, seed)
    kind, r = case["kind"], case["r"]
    if kind in ("adamw", "refresh"):
        left, Gr = s["left"].double(), s["Gr"].double()
        if kind == "refresh":
            return {"P": _orth(left @ (Gr.T @ _normals(seed, case["d_out"], case["k"])))}
        h, P = ADAM, s["P"].double()
        R = Gr @ (P.T @ left).T
        M = h["beta1"] * s["M"].double() + (1 - h["beta1"]) * R
        V = h["beta2"] * s["V"].double() + (1 - h["beta2"]) * R * R
        N = (M / (1 - h["beta1"] ** h["step"])) / (torch.sqrt(V / (1 - h["beta2"] ** h["step"])) + h["eps"])
        W = (1 - h["lr"] * h["weight_decay"]) * s["W"].double() - h["lr"] * h["scale"] * (N @ P.T)
        return {"M": M, "V": V, "W": W}
    X, n = s["X"].double(), case["n"]
    if kind == "qkv":
        S = _normals(seed, n, r)
        Xs, parts = X.T @ S, []
        for W, dY in zip(s["W"], s["dY"]):
            W, dY = W.double(), dY.double()
            Gr = S.T @ dY
            parts.append({"Y": X @ W, "dX": dY @ W.T, "Gr": Gr, "dW": Xs @ Gr})
        return [Xs, parts]
    dY = s["dY"].double()
    if kind == "fp8":
        X8, W8, dY8 = (s[k + "8"].view(torch.float8_e4m3fn).double() * s[k + "_scale"] for k in ("X", "W", "dY"))
        Y, dX = X8 @ W8, dY8 @ W8.T
    else:
        W = s["W"].double().T if kind == "module" else s["W"].double()
        Y, dX = X @ W, dY @ W.T
    if kind == "rsvd" or case.get("compressor") == "rsvd":
        U = _orth(X @ _normals(seed, case["d_in"], r))
        for _ in range(case["power"]):
            U = _orth(X @ _orth(X.T @ U))
    else:
        U = _normals(seed, n, r)
    V, Gr = X.T @ U, U.T @ dY
    out = {"Y": Y, "Xs": V, "dX": dX, "Gr": Gr, "dW": V @ Gr}
    if kind == "rsvd":
        return {"Y": Y, "U": U, "V": V, "dX": dX, "Gr": Gr, "dW": out["dW"]}
    if kind != "module":
        return out
    out = {"Y": Y, "dX": dX, "dW": out["dW"].T}
    if case["bias"]:
        out["Y"], out["dB"] = Y + s["b"].double(), dY.sum(0)
    return out
