"""The dense gradient from its two factors on every kernel that the choice by size takes, with remainders in each dimension: written
and added to C, bfloat16 and float, both orientations.  The three-stage kernel with one, three, four, nine and sixteen K tiles, the
last one masked and (rank 1024) whole: its ring is refilled while the prefetch of C is among the transfers it waits for.

Bound: exact products, fp32 sums of r terms, one rounding of the result: 2^-8 (bfloat16) of the value, 4 2^-24 sqrt(r) (of at
least 256) of the root mean square beside it."""
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


@pytest.mark.parametrize("out_in", [False, True])
@pytest.mark.parametrize("d_in,d_out,r,bf16_c,added,tile", [
    (72, 200, 8, True, False, "64x64"), (1032, 1544, 40, True, False, "128x64"), (2040, 1928, 72, True, False, "128x64"),
    (2568, 2552, 200, True, False, "128x128"), (3064, 8184, 136, True, False, "192x128"), (4088, 4080, 200, True, False, "persistent"),
    (200, 72, 72, True, True, "64x64"), (2056, 2040, 104, True, True, "128x64"), (3064, 2968, 24, True, True, "three-stage"),
    (3064, 2968, 136, True, True, "three-stage"), (3064, 2968, 200, True, True, "three-stage"), (3064, 2968, 520, True, True, "three-stage"),
    (2968, 3064, 1016, True, True, "three-stage"), (2968, 3064, 1024, True, True, "three-stage"), (3064, 2968, 1032, True, True, "192x128"),
    (8200, 6152, 200, True, True, "192x128"), (1032, 1544, 40, False, False, "128x64"), (3080, 8200, 136, False, False, "192x128"),
    (2056, 2040, 104, False, True, "64x64"), (8200, 6152, 200, False, True, "192x128"),
])
def test_dense_gradient(acc, d_in, d_out, r, bf16_c, added, tile, out_in):
    import torch
    dev = "cuda:0"
    M, N = (d_out, d_in) if out_in else (d_in, d_out)
    taken = plan.factor_tile(M, N, r, bf16_c, added)
    assert taken == tile or out_in and tile != "three-stage", taken
    g = torch.Generator(device=dev).manual_seed(r + d_in)
    Xs = torch.randn(d_in, r, generator=g, device=dev).bfloat16()
    Gr = torch.randn(*((d_out, r) if out_in else (r, d_out)), generator=g, device=dev).bfloat16()
    C = torch.randn(M, N, generator=g, device=dev).to(torch.bfloat16 if bf16_c else torch.float32)
    want = Gr.double() @ Xs.double().T if out_in else Xs.double() @ Gr.double()
    want = want + (C.double() if added else 0)
    flags = (acc.ACC_FLAG_W_OUT_IN if out_in else 0) | (acc.ACC_FLAG_DW_ACCUMULATE if added else 0)
    desc = acc.make_desc(1, d_in, d_out, r, flags=flags, dw_dtype=acc.ACC_BF16 if bf16_c else acc.ACC_F32)
    print(f"dW {M} x {N} rank {r} {taken} added={added} bf16={bf16_c}", flush=True)
    acc.acc_linear_dw(desc, Xs, Gr, C)
    rms = want.square().mean().sqrt()
    over = (C.double() - want).abs() - 8 * 4 * 2.0 ** -24 * max(r, 256) ** 0.5 * rms
    assert bool((over <= (2.0 ** -8 * want.abs() if bf16_c else 0)).all())
