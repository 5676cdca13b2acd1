"""GPU parity of the quantizer at the edges of its workgroup tiles (cast pass 128 rows x 256 columns, amax pass 64 rows x 512
columns or more rows of a narrower tensor) and where an amax workgroup takes several pieces, bit for bit against the oracle."""
import pytest

from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import check_quantize

pytestmark = pytest.mark.gpu

RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


# inside one tile; exactly one; a 16-row and a 16-column remainder of a second; several tiles, odd scale rows (unaligned
# scale pieces); tensors so narrow that 2, 8 or 32 lanes of a wavefront span them in the amax pass, with a remainder of its row groups;
# more pieces of its work than workgroups, with few and with many column blocks (272 of them, 530)
@pytest.mark.parametrize("rows,cols", [(112, 240), (128, 256), (144, 272), (656, 784), (32784, 16), (2064, 48), (4112, 176),
                                       (144, 139024), (32, 271120)])
@pytest.mark.parametrize("mode", ["activation", "weight", "gradient", "row_only"])
def test_tile_edges(rows, cols, mode):
    xb = synth.student_t3(rows, cols, 1e-3, rows + cols) if mode == "gradient" else \
        synth.normal_with_outliers(rows, cols, 1.0, rows + cols, frac=0.01)
    xb[-16:, -16:] = 0                                   # an all-zero 16x16 tile: stored scale 0
    xb[-1, 0] = 0x5000                                   # the tensor's largest magnitude in its last row
    if rows * cols > 1 << 22:
        xb[-1, 0], xb[rows // 2, -17] = 0x3f80, 0x5000   # in a column block and a row group that come late
    if mode == "activation":
        check_quantize(xb, RC, rht=True, rht_seed=11)
    elif mode == "weight":
        check_quantize(xb, RC, nv.BLOCK_16x16)
    elif mode == "gradient":
        check_quantize(xb, RC, rounding=nv.ROUND_SR, rht=True, rht_seed=12, sr_seed=13)
    else:
        check_quantize(xb, nv.LAYOUT_ROW)
