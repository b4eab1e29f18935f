"""Which kernel a product of two gradient factors takes, against what the alternatives measured (no GPU needed)."""
import pytest

import plan_util as plan

TILES = ("64x64", "128x64", "128x128", "192x128", "three-stage", "persistent")


# us on an MI355X, in the order of TILES; B [K, N]; the result bfloat16 or float, written or added to C
@pytest.mark.parametrize("m,n,k,bf16_c,added,us", [
    (3072, 1024, 32, True, False, (4.3, 4.4, 4.8, 5.3, None, None)),
    (3584, 3584, 32, True, False, (11.6, 9.5, 9.5, 10.5, None, None)),
    (1024, 8192, 256, True, False, (12.2, 10.4, 9.7, 11.0, None, 13.5)),
    (1536, 3072, 128, True, False, (7.0, 6.0, 6.7, 6.6, None, None)),
    (4096, 4096, 32, True, False, (14.0, 10.8, 10.9, 10.8, None, None)),
    (3072, 3072, 256, True, False, (13.4, 11.0, 12.6, 11.0, None, 13.3)),
    (768, 1544, 192, True, False, (4.8, 4.6, 5.3, 6.2, None, 11.3)),
    (8192, 8192, 128, True, False, (59.5, 62.6, 42.8, 42.0, None, None)),
    (3072, 3072, 32, True, False, (9.1, 7.7, 8.8, 7.4, None, None)),
    (4096, 4096, 256, True, False, (21.6, 16.1, 15.8, 17.1, None, 15.6)),
    (8192, 8192, 256, True, False, (77.9, 92.8, 55.7, 55.9, None, 48.8)),
    (2048, 2048, 256, True, True, (8.0, 8.2, 10.0, 12.0, 12.0, None)),
    (8192, 8192, 128, True, True, (84.2, 99.9, 94.0, 91.1, 80.6, None)),
    (3072, 3072, 64, True, True, (11.1, 10.9, 14.2, 11.6, 10.7, None)),
    (4096, 4096, 64, True, True, (16.1, 16.7, 17.6, 19.1, 18.7, None)),
    (14336, 4096, 64, True, True, (65.2, 72.2, 72.1, 71.9, 59.0, None)),
    (8192, 8192, 256, True, True, (106.8, 116.2, 106.6, 102.0, 117.6, None)),
    (6144, 3072, 256, False, False, (27.3, 20.7, 23.5, 20.4, None, None)),
    (3072, 8192, 256, False, False, (41.1, 33.0, 31.2, 26.5, None, None)),
    (1500, 1500, 32, False, False, (4.9, 5.2, 5.5, 6.2, None, None)),
    (8192, 8192, 32, False, False, (64.8, 65.4, 50.3, 50.6, None, None)),
    (14336, 4096, 128, False, True, (110.4, 124.8, 126.3, 126.1, None, None)),
    (2048, 3072, 256, False, True, (14.1, 12.8, 15.0, 18.6, None, None)),
    (1032, 1544, 128, False, True, (6.4, 7.4, 10.8, 13.8, None, None)),
    (4672, 1792, 32, True, False, (8.3, 7.5, 8.4, 7.2, None, None)), (4096, 2048, 32, True, False, (8.4, 7.2, 6.6, 7.3, None, None)),
    (8192, 1088, 32, True, False, (9.0, 7.7, 8.7, 7.3, None, None)),
    (3072, 3072, 512, True, True, (None, 20.0, None, None, 19.0, None)), (3072, 3072, 1024, True, True, (None, 29.8, None, None, 27.0, None)),
])
def test_factor_product_is_near_the_best(m, n, k, bf16_c, added, us):
    tile = plan.factor_tile(m, n, k, bf16_c, added)
    assert us[TILES.index(tile)] <= 1.14 * min(t for t in us if t), tile
