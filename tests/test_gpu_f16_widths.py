"""GPU parity of the two-pass GEMM's narrower tiles (224, 192 and 160 columns), ragged at both edges, one tile per workgroup
and several as one stream, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(5072, 5072, 1024), (2032, 6128, 2048), (2016, 5088, 2048), (4080, 5104, 1088)])
@pytest.mark.parametrize("per_row", [False, True], ids=["tensor_scale", "row_scales"])
def test_two_pass_widths(M, N, K, per_row):
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
