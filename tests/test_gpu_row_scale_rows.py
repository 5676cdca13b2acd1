"""GPU parity of the row copy with a scale per row on both sides of the lines between a wavefront and a workgroup per row, and of its columns per lane."""
import pytest

from paper_2509_25149_amd import binding as nv, synth
from test_gpu_row_scales import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(16, 1024), (16, 1040), (1024, 1040), (1040, 1040), (1040, 2048), (1040, 2064), (1024, 2048), (48, 4112), (32, 8208), (16, 20496),
                                       (2032, 2064), (2048, 2064), (2048, 2560), (2064, 2576), (2048, 3072), (2048, 3088), (5200, 3072), (5216, 3072)])
@pytest.mark.parametrize("rounding", [nv.ROUND_RNE, nv.ROUND_SR])
def test_rows(rows, cols, rounding):
    xb = synth.normal_with_outliers(rows, cols, 1.0, 1050 + cols, frac=0.01)
    xb[3] = 0
    xb[-1, -1] = 0x5000
    check(xb, nv.LAYOUT_ROW, rounding)
