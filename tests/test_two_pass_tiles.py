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


def test_a_scale_per_row_never_takes_320_rows():
    rng = random.Random(3)
    size = lambda: max(256, int(256 * 80 ** rng.random()) // 16 * 16)
    taken = set()
    for _ in range(3000):
        M, N, K = size(), size(), size() // 64 * 64
        taken.add(tile(M, N, K))
        assert (tile(M, N, K, True) or (0, 0))[0] != 320
    assert taken == {None, (256, 160), (256, 192), (256, 224), (256, 256), (256, 320), (320, 320)}
