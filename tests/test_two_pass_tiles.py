"""Which tile the two-pass GEMM takes (host code only)."""
import os
import random

import pytest

from paper_2509_25149_amd import binding as nv
from test_gemm_routes import TWO_PASS, plan


@pytest.fixture(scope="module", autouse=True)
def library():
    if not os.path.exists(nv.LIB_PATH):
        pytest.skip("libnvfp4_hip.so not built")


def tile(M, N, K, per_row=False):
    """Rows and columns, or None where the product takes another route."""
    route, shape = plan(M, N, K, workspace=True, row_scales=int(per_row))[:2]
    return shape if route == TWO_PASS else None


@pytest.mark.parametrize("M,N,K,takes", [(8192, 20480, 5120, (256, 320)), (8192, 5120, 20480, (256, 320)), (5120, 20480, 8192, (320, 320)),
                                         (5120, 5120, 4096, (320, 320)), (4096, 5120, 5120, (256, 320)), (2048, 5120, 5120, (256, 160)),
                                         (64, 20480, 5120, None)])
def test_products_take_the_tile_whose_rounds_come_out_best(M, N, K, takes):
    assert tile(M, N, K) == takes


# us accumulated in the tile taken / in the larger one of which a round estimate says that it takes less
@pytest.mark.parametrize("M,N,K,takes", [(4928, 12272, 128, (256, 256)),      # 113 / 132
                                         (13312, 1296, 512, (256, 160)),      # 48 / 56
                                         (7088, 12288, 512, (256, 192)),      # 258 / 297
                                         (17904, 1008, 960, (256, 160)),      # 58 / 67
                                         (8448, 2288, 1216, (256, 160)),      # 66 / 74
                                         (8304, 4768, 64, (256, 320)),        # the larger one: 65; 160 columns 73
                                         (7888, 3088, 960, (320, 320)),       # 72; 224 columns 81
                                         (5120, 20480, 512, (320, 320))])     # 315; 256 columns 336
def test_a_larger_tile_has_to_promise_more_where_a_short_contraction_is_accumulated(M, N, K, takes):
    assert plan(M, N, K, accumulate=True, workspace=True, decoded=3)[:2] == (TWO_PASS, takes)
    if K == 512 and M == 7088:
        assert plan(M, N, K, workspace=True, decoded=3)[:2] == (TWO_PASS, (320, 320))


def test_a_scale_per_row_never_takes_320_rows():
    rng = random.Random(3)
    size = lambda: max(256, int(256 * 80 ** rng.random()) // 16 * 16)
    taken = set()
    for _ in range(3000):
        M, N, K = size(), size(), size() // 64 * 64
        taken.add(tile(M, N, K))
        assert (tile(M, N, K, True) or (0, 0))[0] != 320
    assert taken == {None, (256, 160), (256, 192), (256, 224), (256, 256), (256, 320), (320, 320)}
