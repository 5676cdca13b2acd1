"""GPU parity of the bf16 decode without a rotation (8 elements per thread): one rounding of the oracle's FP32 values, at sizes
that fill part of a workgroup, one, and several; per-tensor and per-row tensor scales; padded output rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(16, 16), (32, 64), (48, 80), (272, 1040)])
@pytest.mark.parametrize("per_row", [False, True], ids=["tensor_scale", "row_scales"])
def test_dequantize_bf16(rows, cols, per_row):
    xb = synth.normal_with_outliers(rows, cols, 1.0, 7400 + rows, frac=0.01)
    q = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if per_row else 0))
    ref = oracle.dequantize(oracle.quantize_row_scales(xb, oracle.ROW) if per_row else oracle.quantize(xb, oracle.ROW))
    buf = torch.full((rows, cols + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    nv.nvfp4_dequantize(q, nv.COPY_ROW, out_dtype=nv.OUT_BF16, out=buf[:, :cols])
    got = buf.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :cols], synth.f32_to_bf16_bits(np.asarray(ref, dtype=np.float32)))
    assert np.all(buf[:, cols:].float().cpu().numpy() == 7.0)


def test_more_elements_than_one_launch_holds():
    """2^35 + 2^22 elements (69 GB of bf16): 128 rows repeated 8193 times, so that the small tensor's decode is what repeats."""
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < 120 << 30:
            pytest.skip("needs 90 GB of free GPU memory")
    base, cols, reps = 128, 32768, 8193
    q = nv.nvfp4_quantize(to_dev(synth.normal_with_outliers(base, cols, 1.0, 7500, frac=0.01)), nv.LAYOUT_ROW)
    small = nv.nvfp4_dequantize(q, nv.COPY_ROW, out_dtype=nv.OUT_BF16)
    codes, scales = q.row_codes.repeat(reps, 1), q.row_scales.repeat(reps, 1)
    q.desc.rows, q.desc.row_codes, q.desc.row_scales = base * reps, codes.data_ptr(), scales.data_ptr()
    out = torch.empty((base * reps, cols), dtype=torch.bfloat16, device="cuda")
    nv.nvfp4_dequantize(q, nv.COPY_ROW, out_dtype=nv.OUT_BF16, out=out)
    for r in range(0, reps, 256):
        part = out.view(reps, base, cols)[r:r + 256]
        assert torch.equal(part.view(torch.int16), small.view(torch.int16).expand(part.shape[0], -1, -1)), r
    del out, codes, scales
    torch.cuda.empty_cache()
