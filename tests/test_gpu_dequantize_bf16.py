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
