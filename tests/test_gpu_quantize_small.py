"""GPU parity of the quantizer on both sides of the line between its kernels for small tensors (up to 176 tiles of 128 x 256) and the others, bit for
bit against the oracle: at the edges of a workgroup's 16 x 256 (row copy), 64 x 128 (col copy, amax pass) and 128 x 256 elements."""
import pytest

from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import check_quantize

pytestmark = pytest.mark.gpu
RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


# one block; a remainder of a wavefront's columns; exactly one workgroup and one block more each way; narrower than the amax pass's wavefronts; more
# pieces than its workgroups; 176 tiles; 204, with a remainder each way, which is also with two sets of workgroups for the copies
@pytest.mark.parametrize("rows,cols", [(16, 16), (48, 144), (64, 128), (80, 272), (16, 4112), (4112, 112), (1040, 4112), (2048, 2816), (2064, 2832)])
@pytest.mark.parametrize("mode", ["d0", "d16", "sr_d0", "sr_d16", "row", "sr_row", "col", "sr_col"])
def test_small_tensors(rows, cols, mode):
    sr, which = mode.startswith("sr_"), mode.replace("sr_", "")
    xb = synth.student_t3(rows, cols, 1e-3, rows + cols) if sr else synth.normal_with_outliers(rows, cols, 1.0, rows + cols, frac=0.01)
    xb[-16:, -16:] = 0                                   # an all-zero 16x16 tile: stored scale 0
    xb[-1, 0] = 0x5000                                   # the tensor's largest magnitude in its last row
    kw = dict(rounding=nv.ROUND_SR if sr else nv.ROUND_RNE, sr_seed=17)
    if which == "row":
        check_quantize(xb, nv.LAYOUT_ROW, **kw)
    elif which == "col":
        check_quantize(xb, nv.LAYOUT_COL, rht=True, rht_seed=18, **kw)
    else:
        check_quantize(xb, RC, rht=which == "d16", rht_seed=19, **kw)
