"""GPU parity of the MXFP4 quantizer at the edges of its 128 x 256 tiles, with a set of workgroups per copy (up to 640 tiles, 768 with stochastic rounding) and with one for both."""
import pytest

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_mxfp4 import MODES, RHT_SEED, SR_SEED, assert_mx_copy, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(32, 256), (96, 224), (128, 288), (288, 544), (416, 32), (4128, 5152), (4128, 6176)])
@pytest.mark.parametrize("mode", sorted(MODES))
def test_mx_quantize_tiles(rows, cols, mode):
    m = MODES[mode]
    rounding, rht = m.get("rounding", nv.ROUND_RNE), m.get("rht", False)
    xb = synth.normal_with_outliers(rows, cols, 1.0, 960 + rows, frac=0.01)
    q = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | nv.LAYOUT_COL, nv.BLOCK_MX32, rounding, rht_on_col=rht, rht_seed=RHT_SEED, sr_seed=SR_SEED)
    o_round = oracle.SR if rounding == nv.ROUND_SR else oracle.RNE
    assert_mx_copy(q.row_codes, q.row_scales, oracle.mx_quantize(xb, oracle.ROW, o_round, False, 0, SR_SEED), f"row copy {mode}")
    assert_mx_copy(q.col_codes, q.col_scales, oracle.mx_quantize(xb, oracle.COL, o_round, rht, RHT_SEED, SR_SEED), f"col copy {mode}")
