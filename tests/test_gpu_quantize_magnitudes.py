"""Quantized copies over the whole range of bf16 magnitudes, bit for bit against the oracle: the rotation's power-of-two normalisation is left to the
conversions, so it meets products that are subnormal on one side of it only, clamped encode scales and sums near the largest float."""
import numpy as np
import pytest

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_mxfp4 import assert_mx_copy, to_dev
from test_gpu_rht_sizes import check

pytestmark = pytest.mark.gpu
RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


def scaled(bits, exponent):
    """bf16 bits times 2^exponent, rounded by truncation (subnormal results among them)."""
    v = (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64) * 2.0 ** exponent
    return (v.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)


# 2 tiles: the kernels for small tensors; 204: the others
@pytest.mark.parametrize("rows,cols", [(112, 272), (2064, 2832)])
@pytest.mark.parametrize("d", [2, 4, 16])
@pytest.mark.parametrize("sr", [False, True], ids=["rne", "sr"])
def test_magnitudes(rows, cols, d, sr):
    base = synth.normal_with_outliers(rows, cols, 1.0, rows + d, frac=0.01)
    kw = dict(rounding=nv.ROUND_SR if sr else nv.ROUND_RNE, rht_seed=31 + d, sr_seed=7)
    exponents = (-134, -128, -100, 115) if rows < 1000 else (-128,)   # 115: 16 outliers of 150 sum to less than 2^127
    for e in exponents:
        check(scaled(base, e), d, RC, **kw)
    spread = np.linspace(-130, 100, rows // 16).astype(int).repeat(16)[:, None]       # block rows from the subnormal to the large
    check(scaled(base, spread), d, RC, **kw)


# MXFP4: the block's power of two is the conversions' scale operand, from 2^-127 on (blocks of zeros and subnormals) to 2^125, which only values that are
# not summed reach (all fields that the operand can have: the self-test)
@pytest.mark.parametrize("rows,cols", [(96, 288), (4128, 5152)])
@pytest.mark.parametrize("rht", [False, True], ids=["plain", "rotated"])
@pytest.mark.parametrize("sr", [False, True], ids=["rne", "sr"])
def test_mx_magnitudes(rows, cols, rht, sr):
    base = synth.normal_with_outliers(rows, cols, 1.0, rows, frac=0.01)
    mode = oracle.SR if sr else oracle.RNE
    exponents = (-134, -128, -126, 0, 115) + (() if rht else (120,))      # the largest value, 143 x 2^120, is above 2^127
    for e in exponents if rows < 1000 else (np.linspace(-132, 115, rows // 16).astype(int).repeat(16)[:, None],):
        xb = scaled(base, e)
        xb[:32, :32] = 0
        q = nv.nvfp4_quantize(to_dev(xb), RC, nv.BLOCK_MX32, nv.ROUND_SR if sr else nv.ROUND_RNE, rht_on_col=rht, rht_seed=5, sr_seed=6)
        assert_mx_copy(q.row_codes, q.row_scales, oracle.mx_quantize(xb, oracle.ROW, mode, False, 0, 6), "row copy")
        assert_mx_copy(q.col_codes, q.col_scales, oracle.mx_quantize(xb, oracle.COL, mode, rht, 5, 6), "col copy")
