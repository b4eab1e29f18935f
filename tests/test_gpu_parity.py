"""GPU path vs CPU fp64 oracle through the C ABI, element by element on seeded inputs.

Bar (the benchmark spec): relative Frobenius error <= 1e-2 for bfloat16 outputs, <= 1e-5 for float32, over each whole
output; beside it every 32 x 32 block of every output is held to twice that bar and every element to
|got - want| <= rtol |want| + atol scale (gpu_util.assert_close)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2605_01255_amd import inputs
from oracle import acc_oracle as orc
import gpu_util as gu
import plan_util as plan


@pytest.fixture(scope="module")
def acc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_01255_amd import binding
    return binding


def _check(acc, lin, tol=None, **kw):
    data = inputs.make(lin)
    got = gu.run_layer(acc, lin, data, **kw)
    okw = {k: kw[k] for k in ("want_dw", "row_offset", "seed", "want_db") if k in kw}
    okw["w_out_in"] = bool(kw.get("flags", 0) & acc.ACC_FLAG_W_OUT_IN)
    want = gu.run_oracle(lin, data, **okw)
    code = acc.ACC_BF16 if lin.dtype == "bf16" else acc.ACC_F32
    tol = tol or gu.tolerance(code)
    errs = gu.check_outputs(got, want, tol, lin.name)
    return got, want, errs


def test_c1_fp32(acc):
    """Tiny configuration, float32 end to end: every output within 1e-5."""
    _check(acc, inputs.config("c1")[0])


SHAPES_BF16 = [
    # n, d_in, d_out, r : several tiles plus ragged tails in every dimension
    (512, 512, 768, 64),
    (1000, 512, 640, 8),        # the paper's smallest rank, tuned kernels (surplus sketch columns masked)
    (515, 264, 136, 8),         # the same with K % 64 != 0
    (2049, 1024, 1544, 24),
    (777, 520, 264, 48),
    (1000, 8, 8, 16),
    (3, 64, 72, 16),
    (1, 16, 24, 16),
    (2049, 1032, 1544, 128),
    (4096, 1024, 256, 512),
]


@pytest.mark.parametrize("n,d_in,d_out,r", SHAPES_BF16)
def test_bf16_shapes(acc, n, d_in, d_out, r):
    _check(acc, inputs.Linear(f"bf16_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype="bf16"))


@pytest.mark.parametrize("n,d_in,d_out,r", [(130, 72, 40, 16), (515, 264, 136, 32), (64, 8, 8, 16)])
def test_fp32_shapes(acc, n, d_in, d_out, r):
    _check(acc, inputs.Linear(f"f32_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype="f32", x_kind="plain"))


def test_strided_rows_and_row_offset(acc):
    lin = inputs.Linear("strided", 300, 136, 200, 32, dtype="bf16")
    _check(acc, lin, pad=(8, 16, 24), row_offset=4 * 1000, seed=0x1F00000003)


def test_mixed_factor_and_dw_dtypes(acc):
    lin = inputs.Linear("mixed_bf16", 640, 264, 392, 64, dtype="bf16")
    _check(acc, lin, factor_dtype=0, dw_dtype=0)          # bf16 layer, fp32 factors, fp32 dW
    _check(acc, lin, factor_dtype=1, dw_dtype=0)
    lin32 = inputs.Linear("mixed_f32", 320, 136, 200, 32, dtype="f32", x_kind="plain")
    _check(acc, lin32, factor_dtype=1, dw_dtype=1, tol=1e-2)   # fp32 layer, bf16 factors


def test_outputs_do_not_depend_on_what_they_should_not(acc):
    """Thm 3.2.2(a): dX (and Y) are bitwise independent of seed and rank; runs are repeatable."""
    lin_a = inputs.Linear("indep", 700, 264, 200, 32, dtype="bf16")
    lin_b = inputs.Linear("indep", 700, 264, 200, 64, dtype="bf16")
    data = inputs.make(lin_a)
    a = gu.run_layer(acc, lin_a, data, seed=1)
    b = gu.run_layer(acc, lin_a, data, seed=2)
    c = gu.run_layer(acc, lin_b, data, seed=1)
    a2 = gu.run_layer(acc, lin_a, data, seed=1)
    assert np.array_equal(a["dX"], b["dX"]) and np.array_equal(a["dX"], c["dX"])
    assert np.array_equal(a["Y"], b["Y"]) and np.array_equal(a["Y"], c["Y"])
    assert not np.array_equal(a["Xs"], b["Xs"])
    for k in a:
        assert np.array_equal(a[k], a2[k]), k               # deterministic split-token reduction


def test_skip_sketch_flag_and_no_dw(acc):
    import torch
    lin = inputs.Linear("skip", 256, 72, 104, 16, dtype="bf16")
    data = inputs.make(lin)
    got = gu.run_layer(acc, lin, data, flags=acc.ACC_FLAG_SKIP_SKETCH, want_dw=False)
    assert np.all(got["Xs"] == 7.0)                          # untouched
    want = gu.run_oracle(lin, data, want_dw=False)
    gu.check_outputs(got, want, 1e-2, lin.name, names=("Y", "dX", "Gr"))


def test_factored_gradient_is_unbiased_on_gpu(acc):
    """1000 seeds at the tiny configuration: the mean of dW converges to X^T dY at the predicted rate."""
    import torch
    lin = inputs.config("c1")[0]
    data = inputs.make(lin)
    dev = "cuda:0"
    X, W, dY = (acc.to_device(data[k], dev) for k in ("X", "W", "dY"))
    Y = torch.empty(lin.n, lin.d_out, device=dev)
    Xs = torch.empty(lin.d_in, lin.r, device=dev)
    dX = torch.empty(lin.n, lin.d_in, device=dev)
    Gr = torch.empty(lin.r, lin.d_out, device=dev)
    dW = torch.empty(lin.d_in, lin.d_out, device=dev)
    total = torch.zeros(lin.d_in, lin.d_out, dtype=torch.float64, device=dev)
    Xf, dYf = inputs.as_f64(data["X"]), inputs.as_f64(data["dY"])
    dense = Xf.T @ dYf
    cf = orc.closed_form_variance(Xf, dYf, lin.r)
    sq = 0.0
    ws_f = ws_b = None
    for seed in range(1000):
        desc = acc.make_desc(lin.n, lin.d_in, lin.d_out, lin.r, seed=seed, io_dtype=acc.ACC_F32)
        if ws_f is None:
            ws_f, ws_b = acc.alloc_workspace(desc, False, dev), acc.alloc_workspace(desc, True, dev)
        acc.acc_linear_fwd(desc, X, W, Y, Xs, ws_f)
        acc.acc_linear_bwd(desc, dY, W, Xs, dX, Gr, dW, ws_b)
        total += dW.double()            # torch only accumulates the test statistic
        if seed < 50:
            sq += float(np.sum((dW.double().cpu().numpy() - dense) ** 2))
        if seed + 1 in (10, 100, 1000):
            err = np.linalg.norm(total.cpu().numpy() / (seed + 1) - dense)
            assert 0.9 < err / np.sqrt(cf / (seed + 1)) < 1.1, (seed + 1, err)
    assert abs(sq / 50 / cf - 1.0) < 0.05


FAST_SHAPES = [
    # shapes the tuned bf16 kernels take (K % 64 == 0, r % 64 == 0) with ragged token / column tails
    (1000, 512, 640, 128),      # 128x128 tiles, ragged M
    (4100, 1024, 3080, 256),    # 256x256 tiles, ragged M and N
    (2500, 576, 1096, 64),      # one column slice of the 512 x 64 sketch tile, ragged second channel slab
    (8192, 2048, 2048, 192),    # three column slices
    (33, 64, 64, 64),           # a single stage, partly filled
    (65, 512, 512, 64),         # three stages: both bodies of the unrolled loop and the odd tail
    (4100, 1024, 3080, 32),     # the paper's rank 32: the second column group of the tile is masked
    (20000, 3072, 1024, 16),    # rank 16, 42 token splits over six channel slabs
    (5000, 1536, 520, 96),      # a half-empty last column slice, ragged tokens and channels
    (3000, 512, 1024, 320),     # five column slices per input panel
]


@pytest.mark.parametrize("n,d_in,d_out,r", FAST_SHAPES)
def test_bf16_tuned_kernel_shapes(acc, n, d_in, d_out, r):
    _check(acc, inputs.Linear(f"fast_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype="bf16"))


@pytest.mark.parametrize("d_in,d_out,r", [(64, 3080, 64), (128, 4104, 128), (192, 3080, 192), (256, 3080, 64),
                                          (320, 3080, 64)])
def test_tuned_gemm_with_one_to_five_k_tiles(acc, d_in, d_out, r):
    """Short contractions of a large output, forward K = d_in: one and two K tiles on the ring kernel, three to five on the
    256 x 256 tile, so every combination of its steady-state loop and its two closing K tiles is taken; dense gradient K = r,
    backward K = d_out long."""
    _check(acc, inputs.Linear(f"ktiles_{d_in}x{d_out}_r{r}", 4100, d_in, d_out, r, dtype="bf16"))


@pytest.mark.parametrize("w_oi", [False, True])
def test_operands_beyond_4_gib_take_the_generic_kernels(acc, w_oi):
    """Rows of X (forward) and of dY (backward) so far apart that the operand spans more than 4 GiB, which the tuned products
    and sketch cannot address."""
    import torch
    dev, bf = "cuda:0", torch.bfloat16
    n, d_in, d_out, r, ld = 264, 72, 40, 16, (1 << 23) + 8
    assert n * ld * 2 > 1 << 32
    lin = inputs.Linear("beyond_4_gib", n, d_in, d_out, r, dtype="bf16")
    data = inputs.make(lin)
    want = gu.run_oracle(lin, data)
    flags = acc.ACC_FLAG_W_OUT_IN if w_oi else 0
    W = acc.to_device(np.ascontiguousarray(data["W"].T) if w_oi else data["W"], dev)
    wide = torch.empty(n, ld, dtype=bf, device=dev)

    def spread(a):
        wide[:, :a.shape[1]] = acc.to_device(a, dev)
        wide[:, a.shape[1]:a.shape[1] + 64] = float("nan")
        return wide

    print(f"operands beyond 4 GiB w_oi={w_oi}", flush=True)
    fwd = acc.make_desc(n, d_in, d_out, r, seed=lin.seed, ldx=ld, flags=flags)
    Y, Xs = torch.full((n, d_out), 7.0, dtype=bf, device=dev), torch.full((d_in, r), 7.0, dtype=bf, device=dev)
    acc.acc_linear_fwd(fwd, spread(data["X"]), W, Y, Xs, acc.alloc_workspace(fwd, False, dev))
    bwd = acc.make_desc(n, d_in, d_out, r, seed=lin.seed, ldy=ld, flags=flags)
    dX = torch.full((n, d_in), 7.0, dtype=bf, device=dev)
    Gr = torch.full((d_out, r) if w_oi else (r, d_out), 7.0, dtype=bf, device=dev)
    got = {"Y": acc.to_host_f64(Y), "Xs": acc.to_host_f64(Xs)}
    acc.acc_linear_bwd(bwd, spread(data["dY"]), W, None, dX, Gr, None, acc.alloc_workspace(bwd, True, dev))
    got.update(dX=acc.to_host_f64(dX), Gr=acc.to_host_f64(Gr).T if w_oi else acc.to_host_f64(Gr))
    gu.check_outputs(got, {k: want[k] for k in got}, 1e-2, lin.name)


def test_tuned_kernels_fp32_dw_and_strides(acc):
    lin = inputs.Linear("fast_strided", 1500, 512, 768, 128, dtype="bf16")
    _check(acc, lin, dw_dtype=0, pad=(64, 8, 72), row_offset=4 * 77, seed=0xABCDEF0123)


def test_big_tile_gemm_with_strides(acc):
    """256 x 256 tiles (the epilogue runs inside the last K tile and stores through a buffer resource) on strided
    X / dX, W and Y / dY with ragged M and N: the padding columns of Y and dX keep their contents."""
    lin = inputs.Linear("big_strided", 4100, 1024, 3080, 128, dtype="bf16")
    _check(acc, lin, pad=(40, 8, 24))


@pytest.mark.parametrize("n,d_in,d_out,r,pad", [
    (16284, 192, 3072, 64, (0, 0, 0)),      # forward: three K tiles (the minimum), ragged last row of tiles
    (16384, 256, 3072, 64, (64, 8, 24)),    # four K tiles (stage parity unchanged from tile to tile), strided
    (16384, 320, 3072, 64, (0, 0, 0)),      # five K tiles (stage parity alternates)
    (16384, 3072, 3136, 64, (0, 0, 0)),     # backward: 49 K tiles, three output tiles per work-group
    (2304, 256, 13560, 64, (0, 0, 0)),      # 9 x 53 tiles in a map of 1024 slots: empty slots between a work-group's tiles
])
def test_persistent_gemm_across_output_tiles(acc, n, d_in, d_out, r, pad):
    """More than 256 slots in the map of 256 x 256 output tiles: 256 persistent work-groups whose K pipeline
    runs across the tile boundary (next tile requested inside the last K tiles of the one before)."""
    assert "256x256" in (plan.gemm_tile(n, d_out, d_in)[0], plan.gemm_tile(n, d_in, d_out)[0])
    _check(acc, inputs.Linear(f"persist_{n}x{d_in}x{d_out}", n, d_in, d_out, r, dtype="bf16"), pad=pad)


def _seeded_big_shapes(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        n = int(rng.integers(3000, 9000))
        d_in = 8 * int(rng.integers(24, 160))        # 192 ... 1272; at K % 64 != 0 the last K tile is masked
        d_out = 8 * int(rng.integers(380, 640))      # 3040 ... 5112
        if rng.integers(0, 3):
            d_in = 64 * max(3, d_in // 64)           # mostly multiples of 64
        r = int(rng.choice([16, 32, 64, 128, 192, 256]))
        if -(-n // 256) * -(-d_out // 256) >= 192:
            out.append((n, d_in, d_out, r))
    return out


@pytest.mark.parametrize("n,d_in,d_out,r", _seeded_big_shapes(6, 2024))
def test_seeded_random_shapes_on_the_large_tile_kernels(acc, n, d_in, d_out, r):
    """Seeded random sizes with at least 192 output tiles of 256 x 256 in the forward product (ragged in every
    dimension): whatever kernels the planner picks, every output meets the full bar."""
    _check(acc, inputs.Linear(f"rand_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype="bf16"))


def test_one_launch_flag_gives_identical_results(acc):
    """ACC_FLAG_ONE_LAUNCH interleaves GEMM and sketch work-groups in one grid: same outputs, bit for bit
    for the exact products, within tolerance of the oracle for the factors."""
    lin = inputs.Linear("one_launch", 4100, 1024, 3080, 256, dtype="bf16")
    data = inputs.make(lin)
    two = gu.run_layer(acc, lin, data)
    one = gu.run_layer(acc, lin, data, flags=acc.ACC_FLAG_ONE_LAUNCH)
    assert np.array_equal(one["Y"], two["Y"]) and np.array_equal(one["dX"], two["dX"])
    want = gu.run_oracle(lin, data)
    gu.check_outputs(one, want, 1e-2, lin.name + " one launch")


# ---- the paper's weight orientation ([d_out, d_in], Def. 3.1) and the bias gradient ------------------
@pytest.mark.parametrize("n,d_in,d_out,r,dtype", [
    (130, 72, 40, 16, "f32"),          # float32 kernel
    (777, 520, 264, 48, "bf16"),       # ring kernel, last K tile masked
    (1000, 512, 640, 128, "bf16"),     # one round of small tiles
    (4100, 1024, 3080, 256, "bf16"),   # large tiles, ragged M and N
    (2500, 576, 1096, 64, "bf16"),     # one column slice of the sketch tile, ragged channel slab
])
def test_weight_out_in_orientation_and_bias_gradient(acc, n, d_in, d_out, r, dtype):
    lin = inputs.Linear(f"oi_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype=dtype)
    got, want, _ = _check(acc, lin, flags=acc.ACC_FLAG_W_OUT_IN, want_db=True)
    assert got["Gr"].shape == (d_out, r) and got["dW"].shape == (d_out, d_in) and got["dB"].shape == (d_out,)
    # same layer in the default orientation: exact products bit for bit, factors transposed bit for bit
    ref = gu.run_layer(acc, lin, inputs.make(lin))
    assert np.array_equal(got["Y"], ref["Y"]) and np.array_equal(got["dX"], ref["dX"])
    assert np.array_equal(got["Xs"], ref["Xs"]) and np.array_equal(got["Gr"], ref["Gr"].T)


def test_weight_out_in_with_strides_and_fp32_dw(acc):
    lin = inputs.Linear("oi_strided", 1500, 512, 768, 128, dtype="bf16")
    _check(acc, lin, flags=acc.ACC_FLAG_W_OUT_IN, dw_dtype=0, pad=(64, 8, 72), row_offset=4 * 77,
           seed=0xABCDEF0123, want_db=True)


@pytest.mark.parametrize("n,d_out,dtype", [(1, 8, "bf16"), (5, 24, "f32"), (1000, 520, "bf16"),
                                           (16384, 3072, "bf16"), (4099, 264, "f32")])
def test_bias_gradient_shapes(acc, n, d_out, dtype):
    """dB = column sums of dY, fp32 accumulation; bitwise reproducible."""
    lin = inputs.Linear(f"db_{n}x{d_out}", n, 16, d_out, 16, dtype=dtype)
    data = inputs.make(lin)
    a = gu.run_layer(acc, lin, data, want_dw=False, want_db=True, dw_dtype=0)
    b = gu.run_layer(acc, lin, data, want_dw=False, want_db=True, dw_dtype=0)
    want = orc.bias_grad(inputs.as_f64(data["dY"]))
    assert np.array_equal(a["dB"], b["dB"])
    # fp32 summation in a fixed tree: at most 16 rows per wave, 16 waves, then 16 + 4 partials -> at most
    # 50 additions on any path for n <= 16384, so |error| <= 50 * 2^-24 * sum|dY| < 1e-5 * sum|dY| per column
    scale = np.sum(np.abs(inputs.as_f64(data["dY"])), axis=0)
    assert np.all(np.abs(a["dB"] - want) <= 1e-5 * scale + 1e-30), np.max(np.abs(a["dB"] - want) / (scale + 1e-30))


@pytest.mark.parametrize("dw_dtype,shape", [(0, (1000, 512, 640, 128)), (1, (1000, 512, 640, 128)),
                                            (0, (130, 72, 40, 16)), (0, (4100, 1024, 3080, 256))])
def test_dense_gradient_accumulates_over_micro_batches(acc, dw_dtype, shape):
    """ACC_FLAG_DW_ACCUMULATE: two micro-batches (different data and seeds) summed into one dense dW."""
    import torch
    n, d_in, d_out, r = shape
    dtype = "bf16" if d_in % 64 == 0 else "f32"
    code = acc.ACC_BF16 if dtype == "bf16" else acc.ACC_F32
    dcode = dw_dtype if dtype == "bf16" else acc.ACC_F32
    dW = torch.zeros(d_in, d_out, dtype=acc.torch_dtype(dcode), device="cuda:0")
    want = None
    for mb, seed in enumerate((11, 12)):
        lin = inputs.Linear(f"acc{mb}", n, d_in, d_out, r, dtype=dtype, seed=seed)
        data = inputs.make(lin)
        if mb:  # a different micro-batch: reverse the token order of the first one's data
            data = {k: (np.ascontiguousarray(v[::-1]) if k in ("X", "dY") else v) for k, v in data.items()}
        X, W, dY = (acc.to_device(data[k]) for k in ("X", "W", "dY"))
        fd = acc.make_desc(n, d_in, d_out, r, seed=seed, io_dtype=code, dw_dtype=dcode)
        bd = acc.make_desc(n, d_in, d_out, r, seed=seed, io_dtype=code, dw_dtype=dcode,
                           flags=acc.ACC_FLAG_DW_ACCUMULATE if mb else 0)
        Y = torch.empty(n, d_out, dtype=acc.torch_dtype(code), device="cuda:0")
        dX = torch.empty(n, d_in, dtype=acc.torch_dtype(code), device="cuda:0")
        Xs = torch.empty(d_in, r, dtype=acc.torch_dtype(code), device="cuda:0")
        Gr = torch.empty(r, d_out, dtype=acc.torch_dtype(code), device="cuda:0")
        acc.acc_linear_fwd(fd, X, W, Y, Xs, acc.alloc_workspace(fd, False))
        acc.acc_linear_bwd(bd, dY, W, Xs, dX, Gr, dW, acc.alloc_workspace(bd, True))
        Xf, Wf, dYf = (inputs.as_f64(data[k]) for k in ("X", "W", "dY"))
        S = orc.sketch_matrix(seed, n, r)
        _, Xs_o = orc.linear_fwd(Xf, Wf, S=S)
        _, _, want = orc.linear_bwd(dYf, Wf, Xs_o, S=S, dW_prev=want)
    torch.cuda.synchronize()
    # bf16 factors bound the error even for a float dW
    gu.check_outputs({"dW": acc.to_host_f64(dW)}, {"dW": want}, 1e-2 if dtype == "bf16" else 1e-5, "accumulated")


def test_calls_can_be_captured_in_a_hip_graph_and_replayed(acc):
    """The library only enqueues kernels on the caller's stream (no allocation, no memset, no sync), so a
    forward + backward + bias gradient can be captured once and replayed; every replay must reproduce the
    eager result bit for bit, with eager work and synchronisations between replays."""
    import torch
    lin = inputs.Linear("graph", 4100, 1024, 3080, 256, dtype="bf16")
    data = inputs.make(lin)
    X, W, dY = (acc.to_device(data[k]) for k in ("X", "W", "dY"))
    desc = acc.make_desc(lin.n, lin.d_in, lin.d_out, lin.r, seed=5, io_dtype=acc.ACC_BF16)
    bf = torch.bfloat16
    outs = {k: torch.empty(*shp, dtype=bf, device="cuda:0") for k, shp in
            (("Y", (lin.n, lin.d_out)), ("dX", (lin.n, lin.d_in)), ("Xs", (lin.d_in, lin.r)),
             ("Gr", (lin.r, lin.d_out)), ("dW", (lin.d_in, lin.d_out)), ("dB", (lin.d_out,)))}
    ws_f, ws_b = acc.alloc_workspace(desc, False), acc.alloc_workspace(desc, True)

    def enqueue():
        acc.acc_linear_fwd(desc, X, W, outs["Y"], outs["Xs"], ws_f)
        acc.acc_linear_bwd(desc, dY, W, outs["Xs"], outs["dX"], outs["Gr"], outs["dW"], ws_b)
        acc.acc_linear_bias_grad(desc, dY, outs["dB"], ws_b)

    enqueue()                      # eager: also raises the kernels' LDS limits outside the capture
    torch.cuda.synchronize()
    eager = {k: v.clone() for k, v in outs.items()}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            enqueue()
    torch.cuda.synchronize()
    for rep in range(3):
        for v in outs.values():
            v.fill_(3.0)           # eager work between replays; also proves the replay rewrites everything
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in outs:
            assert torch.equal(outs[k], eager[k]), (rep, k)


@pytest.mark.parametrize("n,d_in,d_out,r,dtype,one_launch", [
    (1000, 512, 640, 128, "bf16", False),   # 512 x 64 sketch tile
    (1000, 512, 640, 128, "bf16", True),    # the 512 x 128 tile that the one-launch flag selects
    (777, 520, 264, 48, "bf16", False),     # surplus sketch columns masked
    (700, 72, 40, 16, "f32", False),        # float32 kernel
])
def test_row_offsets_crossing_2_pow_34(acc, n, d_in, d_out, r, dtype, one_launch):
    """A shard whose global token indices cross 2^34: the high bits move into the fourth counter word."""
    lin = inputs.Linear(f"hi_offset_{n}x{d_in}x{d_out}_r{r}", n, d_in, d_out, r, dtype=dtype, seed=0x5EED5EED5EED)
    _check(acc, lin, row_offset=(1 << 34) - 512, flags=acc.ACC_FLAG_ONE_LAUNCH if one_launch else 0)


def test_all_zero_inputs_give_exact_zeros(acc):
    """Degenerate inputs: X = 0 (then Y, Xs, dW are exactly 0) and dY = 0 (then dX, Gr, dW, dB are exactly 0)."""
    lin = inputs.Linear("zeros", 1000, 512, 640, 128, dtype="bf16")
    data = inputs.make(lin)
    zx = dict(data, X=np.zeros_like(data["X"]))
    got = gu.run_layer(acc, lin, zx)
    for key in ("Y", "Xs", "dW"):
        assert np.all(got[key] == 0.0), key
    zg = dict(data, dY=np.zeros_like(data["dY"]))
    got = gu.run_layer(acc, lin, zg, want_db=True)
    for key in ("dX", "Gr", "dW", "dB"):
        assert np.all(got[key] == 0.0), key


def test_concurrent_host_threads_on_their_own_streams(acc):
    """The library keeps no state between calls: two host threads, each with its own stream, buffers and workspace,
    call it at the same time (ctypes releases the interpreter lock during a call) and must reproduce, bit for bit,
    what the same calls give one after the other."""
    import threading
    import torch
    dev = "cuda:0"
    lins = [inputs.Linear("thr0", 2100, 1024, 1544, 128, dtype="bf16", seed=11),
            inputs.Linear("thr1", 1800, 1544, 1024, 64, dtype="bf16", seed=12)]
    jobs = []
    for lin in lins:
        data = inputs.make(lin)
        X, W, dY = (acc.to_device(data[k], dev) for k in ("X", "W", "dY"))
        desc = acc.make_desc(lin.n, lin.d_in, lin.d_out, lin.r, seed=lin.seed)
        bf = torch.bfloat16
        outs = {k: torch.empty(*shp, dtype=bf, device=dev) for k, shp in
                (("Y", (lin.n, lin.d_out)), ("dX", (lin.n, lin.d_in)), ("Xs", (lin.d_in, lin.r)),
                 ("Gr", (lin.r, lin.d_out)), ("dW", (lin.d_in, lin.d_out)))}
        jobs.append(dict(desc=desc, X=X, W=W, dY=dY, outs=outs, ws_f=acc.alloc_workspace(desc, False, dev),
                         ws_b=acc.alloc_workspace(desc, True, dev), stream=torch.cuda.Stream()))

    def run(job, reps):
        for _ in range(reps):
            o = job["outs"]
            acc.acc_linear_fwd(job["desc"], job["X"], job["W"], o["Y"], o["Xs"], job["ws_f"], stream=job["stream"])
            acc.acc_linear_bwd(job["desc"], job["dY"], job["W"], o["Xs"], o["dX"], o["Gr"], o["dW"], job["ws_b"],
                               stream=job["stream"])

    for job in jobs:            # serial reference
        run(job, 1)
    torch.cuda.synchronize()
    ref = [{k: v.clone() for k, v in job["outs"].items()} for job in jobs]
    for job in jobs:
        for v in job["outs"].values():
            v.fill_(3.0)
    torch.cuda.synchronize()
    errors = []

    def worker(job):
        try:
            run(job, 20)
        except Exception as e:   # surfaces in the main thread below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(job,)) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for job, r in zip(jobs, ref):
        for k in r:
            assert torch.equal(job["outs"][k], r[k]), k
