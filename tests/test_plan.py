"""The choices by size that the library makes on the host, against what the alternatives measured (no GPU needed)."""
import pytest

import plan_util as plan

TILES = ("128x64", "64x64", "64x32", "32x32")


# us on an MI355X, in the order of TILES; A [M, K] and B [K, N] with their rows contiguous
@pytest.mark.parametrize("m,n,k,us", [
    (2048, 2048, 1024, (72.3, 76.7, 84.3, 87.6)),
    (2048, 1024, 2048, (72.6, 72.4, 103.1, 86.4)),
    (300, 4096, 2048, (71.3, 71.2, 56.4, 58.9)),
    (2504, 1000, 3000, (185.7, 198.3, 158.3, 163.6)),
    (256, 512, 256, (12.1, 8.1, 6.0, 5.1)),
    (3656, 280, 288, (14.1, 13.8, 12.0, 12.8)),
    (3072, 1024, 3072, (190.0, 203.0, 166.0, 194.2)),
    (2052, 2056, 1032, (106.2, 95.0, 87.6, 96.6)),
    (1032, 1032, 520, (22.7, 22.1, 18.4, 19.8)),
    (2044, 2040, 1000, (68.2, 74.4, 83.0, 89.4)),
    (400, 8000, 600, (42.5, 45.2, 47.0, 45.5)),
    (4096, 4096, 1024, (260.5, 281.8, 303.1, 352.4)),
    (600, 600, 4096, (138.0, 83.8, 52.8, 53.5)),
    (704, 1504, 1000, (38.2, 38.1, 30.6, 32.6)),
    (3000, 3000, 1000, (167.9, 161.3, 166.6, 194.9)),
    (384, 3072, 3072, (105.3, 107.1, 83.9, 88.1)),
    (1024, 64, 4096, (139.0, 82.5, 51.7, 39.5)),
    (1536, 1024, 2048, (71.7, 71.6, 56.8, 66.8)),
    (2337, 2496, 1472, (138.1, 158.8, 156.4, 166.9)), (2500, 2304, 1024, (95.9, 110.8, 101.8, 117.1)), (2453, 2304, 1408, (132.3, 144.7, 138.9, 152.8)),
    (2236, 2240, 640, (62.0, 53.5, 57.2, 65.8)),   # 2.5 of 128 x 64 to a compute unit, five of 64 x 64, all resident
])
def test_float32_tile_is_near_the_best(m, n, k, us):
    tile = plan.f32_tile(m, n)
    assert us[TILES.index(tile)] <= 1.12 * min(us), tile


# us of a product on 32 x 32 tiles with two stages and with four
@pytest.mark.parametrize("m,n,k,two,four", [
    (405, 1728, 3392, 60.3, 58.2), (531, 1280, 2432, 43.7, 42.6), (391, 2392, 1472, 35.0, 34.0), (339, 2112, 1536, 30.1, 29.6),
    (726, 1024, 384, 9.6, 9.8), (873, 832, 720, 15.8, 16.1), (1463, 448, 576, 12.6, 12.8), (448, 1176, 392, 10.1, 10.3), (913, 640, 3056, 55.7, 54.4),
])
def test_stages_of_32_x_32_tiles(m, n, k, two, four):
    assert plan.f32_tile(m, n) == "32x32"
    assert (four if plan.f32_four_stages(m, n, k) else two) <= 1.02 * min(two, four)


# us of the sketch with a stored S and with the generic kernel, tokens x channels at rank
@pytest.mark.parametrize("n,channels,r,stored,generic", [
    (8192, 256, 16, 78.3, 30.7), (8192, 256, 64, 80.1, 34.1), (8192, 256, 256, 84.8, 44.7), (7000, 256, 64, 69.1, 32.8),
    (6000, 256, 64, 60.0, 31.3), (4096, 256, 16, 41.4, 27.3), (4096, 256, 64, 42.3, 28.9), (4096, 256, 256, 46.4, 30.0),
    (2048, 256, 64, 23.6, 26.6), (1024, 256, 64, 14.2, 25.3), (12288, 384, 64, 116.0, 56.8), (16384, 512, 16, 150.2, 70.6),
    (16384, 512, 64, 151.6, 69.8), (16384, 512, 256, 157.3, 106.9), (14000, 512, 64, 40.2, 62.3), (8192, 512, 64, 19.6, 41.3),
    (4096, 512, 64, 14.7, 29.3), (32768, 1024, 64, 300.0, 153.1), (30000, 1024, 64, 142.8, 144.0), (24000, 1024, 64, 63.0, 118.2),
    (16384, 1024, 64, 45.4, 85.2), (65536, 2048, 32, 586.0, 449.4), (60000, 2048, 32, 263.5, 402.4), (50000, 2048, 32, 116.6, 336.8),
    (2048, 1024, 64, 12.9, 26.9), (4096, 1024, 256, 45.2, 59.5), (4096, 4096, 256, 93.4, 193.9), (2048, 2048, 64, 16.9, 39.2),
    (256, 256, 16, 7.0, 24.0), (1500, 256, 128, 19.2, 25.9), (3000, 256, 256, 35.3, 28.2)])
def test_float32_sketch_takes_the_faster_form(n, channels, r, stored, generic):
    takes_stored = plan.f32_sketch_splits(n, channels, r) > 0
    assert (stored if takes_stored else generic) <= 1.05 * min(stored, generic)


# us of a float32 forward pass whose sketch and exact product share a launch, and of one where they do not
@pytest.mark.parametrize("n,d_in,d_out,r,shared,apart", [
    (256, 256, 512, 16, 7.4, 11.8), (256, 512, 2624, 16, 14.9, 19.1), (1024, 384, 768, 64, 18.0, 23.5),
    (2624, 384, 256, 128, 19.6, 24.2), (256, 3072, 384, 256, 36.7, 40.2), (1024, 3072, 256, 256, 45.8, 52.9), (256, 3072, 3072, 64, 56.6, 59.9),
    (1500, 512, 512, 128, 20.8, 24.8), (300, 3072, 768, 16, 34.5, 38.6), (854, 2656, 896, 256, 60.5, 66.6),
    (512, 3072, 1536, 256, 60.3, 65.5),
])
def test_float32_products_share_a_launch_where_that_is_faster(n, d_in, d_out, r, shared, apart):
    assert (plan.f32_pair(n, d_in, d_out, r) > 0) == (shared < apart)


def test_stored_sketch_fits_the_workspace():
    for n in (1, 31, 255, 256, 1000, 4096, 9999, 65536, 130001):
        for channels in (8, 40, 256, 520, 2048, 14336):
            for r in (8, 24, 64, 264, 512):
                for f32_factor in (True, False):
                    assert plan.f32_sketch_fits(n, channels, r, f32_factor), (n, channels, r, f32_factor)


def test_raised_lds_limits_are_remembered_for_every_kernel_and_device():
    """A launch whose kernel is not in the table sets the limit again."""
    assert plan.lib().raised_lost(plan.lib().raised_capacity(), 64) == 0


# us of a forward pass with 1024 outputs: the token splits of 512 channels, and the splits and slabs chosen
@pytest.mark.parametrize("n,channels,r,slab,two_sums,before,now", [
    (4096, 4096, 128, 256, True, 56.1, 52.3), (2048, 4096, 256, 256, True, 46.8, 41.8), (600, 8192, 256, 256, True, 53.0, 49.6),
    (1500, 5120, 256, 256, True, 52.1, 46.0), (16384, 4096, 64, 512, False, 129.3, 129.3), (4096, 1024, 256, 128, True, 27.1, 26.0),
    (4096, 3072, 256, 512, False, 48.8, 48.8), (2500, 2048, 256, 512, False, 34.4, 34.4), (6000, 3072, 256, 512, False, 60.8, 60.8),
    (4096, 3584, 256, 512, False, 53.4, 53.4), (2049, 3072, 512, 512, False, 55.9, 55.9),
    (21418, 448, 384, 512, False, 38.6, 38.6), (15018, 2208, 128, 512, False, 75.0, 75.0), (13453, 448, 512, 512, False, 44.3, 44.3),
    (23571, 488, 256, 512, False, 48.3, 48.3), (7950, 4480, 128, 512, False, 45.0, 45.0),
])
def test_sketch_splits_are_near_the_best(n, channels, r, slab, two_sums, before, now):
    p = plan.sketch(n, channels, r)
    assert (p.slab, p.two_sums) == (slab, two_sums)
    assert now <= 1.02 * before


def test_sketch_splits_fit_the_workspace_and_the_chip():
    """Never more splits than the workspace holds, never more work-groups than compute units where 512 channels made no more; no
    running sum longer than one of the splits that 512 channels make, and those splits themselves with a float factor."""
    for n in (1, 31, 257, 300, 700, 1030, 2049, 4096, 4097, 16384, 21418, 65536):
        for channels in (8, 128, 136, 448, 520, 1024, 3072, 3080, 8192, 14336, 40000):
            for r in (8, 64, 72, 256, 384, 512):
                columns = -(-r // 64)
                most = max(1, min(256 // (-(-channels // 512) * columns), -(-n // 256), 64))
                tokens = -(--(-n // most) // 32) * 32
                for bf16_factor in (True, False):
                    p = plan.sketch(n, channels, r, bf16_factor)
                    if not p.tuned or p.columns == 128:
                        continue
                    assert p.slab in (128, 256, 512) and p.tokens % 32 == 0
                    assert p.splits == -(-n // p.tokens) <= p.room == -(-n // tokens)
                    assert p.tiles * p.splits <= max(256, -(-channels // 512) * columns)
                    if p.slab < 512:   # a die takes whole pairs of slab and split, with all their column slices, on 32 compute units
                        assert -(-p.tiles // columns * p.splits // 8) * columns <= 32
                    assert -(-p.tokens // 32 // (2 if p.two_sums else 1)) * 32 <= tokens
                    assert bf16_factor or (p.tokens == tokens and not p.two_sums)
