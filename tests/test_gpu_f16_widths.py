"""GPU parity of the two-pass GEMM's narrower tiles (224, 192 and 160 columns), ragged at both edges, one tile per workgroup
and several as one stream, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import TWO_PASS, plan
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


# the last three: more tiles than CUs
@pytest.mark.parametrize("M,N,K,columns", [(5408, 2192, 320, 224), (2736, 4368, 256, 192), (4624, 1680, 1088, 160), (6160, 3984, 256, 224), (6112, 3984, 256, 192),
                                           (6432, 7728, 320, 160)])
@pytest.mark.parametrize("per_row", [False, True], ids=["tensor_scale", "row_scales"])
def test_two_pass_widths(M, N, K, columns, per_row):
    assert plan(M, N, K, workspace=True, row_scales=int(per_row))[:2] == (TWO_PASS, (256, columns))
    xb, wb = synth.normal_with_outliers(M, K, 1.0, 7200 + K, frac=0.01), synth.normal(N, K, 0.02, 7300 + N)
    qx = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if per_row else 0))
    qw = nv.nvfp4_quantize(to_dev(wb), nv.LAYOUT_ROW)
    rx = oracle.quantize_row_scales(xb, oracle.ROW) if per_row else oracle.quantize(xb, oracle.ROW)
    ref = oracle.gemm_f64(rx, oracle.quantize(wb, oracle.ROW))
    ws = torch.empty(nv.gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, out=buf[:, :N], workspace=ws)
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)                 # nothing stored past a row's last column
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    y16 = nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_BF16, workspace=ws)
    assert torch.equal(y16, buf[:, :N].to(torch.bfloat16))
    acc = buf[:, :N].clone()
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_F32_ACCUMULATE, out=acc, workspace=ws)
    assert torch.equal(acc, buf[:, :N] + buf[:, :N])
