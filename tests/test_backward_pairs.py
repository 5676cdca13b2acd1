"""Which backward passes run their two products in one launch (host code only)."""
import ctypes
import os

import pytest

from paper_2509_25149_amd import binding as nv


@pytest.fixture(scope="module", autouse=True)
def library():
    if not os.path.exists(nv.LIB_PATH):
        pytest.skip("libnvfp4_hip.so not built")


def one_launch(tokens, d_in, d_out):
    i64 = ctypes.c_int64
    workspace = max(nv.linear_workspace_bytes(tokens, d_in, d_out), 256)
    return bool(nv.load_library().nvfp4_internal_backward_pairs(i64(tokens), i64(d_in), i64(d_out), ctypes.c_size_t(workspace)))


# us in one launch / two
@pytest.mark.parametrize("t,d_in,d_out", [(4416, 384, 9456),     # 195 / 176
                                          (5216, 320, 10752), (2672, 368, 19792),
                                          (2048, 960, 3600),     # 70 / 65
                                          (3408, 960, 6768),     # 201 / 192
                                          (2032, 3168, 1088), (1328, 576, 11840)])
def test_products_that_come_out_even_apart_stay_apart(t, d_in, d_out):
    assert not one_launch(t, d_in, d_out)


@pytest.mark.parametrize("t,d_in,d_out", [(1040, 2064, 1296),    # 37 / 42
                                          (416, 1280, 512), (240, 2304, 16384),
                                          (192, 4096, 1280),     # 20 / 26
                                          (1200, 480, 12512),    # 83 / 95
                                          (4992, 832, 7216), (6912, 448, 13664), (5504, 3328, 256)])
def test_products_that_leave_places_empty_share_a_launch(t, d_in, d_out):
    assert one_launch(t, d_in, d_out)


def test_larger_products_do_not():
    assert not one_launch(8192, 5120, 20480) and not one_launch(4096, 5120, 5120)
