"""How the cast pass of the quantizer goes over memory (host code only): from the end 1, in bands 2, in strips 4."""
import ctypes
import os

import pytest

from paper_2509_25149_amd import binding as nv

RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


@pytest.mark.skipif(not os.path.exists(nv.LIB_PATH), reason="libnvfp4_hip.so not built")
@pytest.mark.parametrize("rows,cols,layout,walk", [
    (8192, 5120, RC, 4), (5120, 20480, RC, 1 | 4), (8192, 16384, RC, 1 | 4), (8192, 20480, RC, 0),      # aligned: both copies up to 256 MB
    (8192, 20480, nv.LAYOUT_ROW, 4), (8192, 20480, nv.LAYOUT_COL, 4),                                    # one copy of any size
    (8208, 16400, RC, 1 | 4), (8176, 19504, RC, 4), (2064, 2832, nv.LAYOUT_ROW, 2), (272, 131088, nv.LAYOUT_ROW, 4)])   # rows anywhere
def test_walk(rows, cols, layout, walk):
    out, i64 = (ctypes.c_int * 5)(), ctypes.c_int64
    nv.load_library().nvfp4_internal_quantize_plan(i64(rows), i64(cols), layout & nv.LAYOUT_ROW, layout & nv.LAYOUT_COL, 0, 0, out)
    assert out[2] == walk


SR, GIVEN = 2, 4   # stochastic rounding; the amax given


# Aligned tensors that take longer in strips than along their rows: one copy whose amax is given, a tall col copy somewhat larger than the memory-side cache
@pytest.mark.skipif(not os.path.exists(nv.LIB_PATH), reason="libnvfp4_hip.so not built")
@pytest.mark.parametrize("rows,cols,layout,options,walk", [
    (9216, 19968, nv.LAYOUT_ROW, GIVEN, 0), (3840, 65792, nv.LAYOUT_ROW, GIVEN | SR, 0), (8192, 16384, nv.LAYOUT_ROW, GIVEN, 4), (8192, 16384, nv.LAYOUT_ROW, GIVEN | SR, 0),
    (13312, 6144, nv.LAYOUT_COL, GIVEN, 0), (13312, 6400, nv.LAYOUT_COL, GIVEN, 4), (8192, 20480, nv.LAYOUT_COL, GIVEN, 4), (13312, 6144, RC, GIVEN, 4),
    (8192, 20480, RC, GIVEN, 0), (79616, 2048, nv.LAYOUT_COL, 0, 0), (14080, 12288, nv.LAYOUT_COL, 0, 0), (13792, 12160, nv.LAYOUT_COL, 0, 0),
    (19456, 9984, nv.LAYOUT_COL, 0, 4), (19456, 9984, nv.LAYOUT_COL, SR, 0), (39680, 3840, nv.LAYOUT_COL, SR, 0), (39680, 3840, nv.LAYOUT_COL, 0, 4),
    (12288, 14080, nv.LAYOUT_COL, 0, 4), (65536, 2048, nv.LAYOUT_COL, 0, 1 | 4), (102400, 2048, nv.LAYOUT_COL, 0, 4)])
def test_walk_of_tensors_that_strips_slow_down(rows, cols, layout, options, walk):
    out, i64 = (ctypes.c_int * 5)(), ctypes.c_int64
    nv.load_library().nvfp4_internal_quantize_plan(i64(rows), i64(cols), layout & nv.LAYOUT_ROW, layout & nv.LAYOUT_COL, 0, options, out)
    assert out[2] == walk
