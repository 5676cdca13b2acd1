"""GPU parity of the two-pass GEMM in each of its tiles, ragged at both edges, one tile per workgroup and several as one stream, against
the oracle's binary64 product."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


def tile(M, N, K, per_row):
    out = (ctypes.c_int * 2)()
    i64 = ctypes.c_int64
    assert nv.load_library().nvfp4_internal_two_pass_tile(i64(M), i64(N), i64(K), int(per_row), ctypes.c_size_t(nv.gemm_workspace_bytes(M, N, K)), out)
    return tuple(out)


@pytest.mark.parametrize("M,N,K,per_row,takes", [
    (3088, 6176, 256, False, (320, 320)), (4112, 9664, 256, False, (320, 320)), (2096, 19184, 320, False, (320, 320)),
    (1216, 13152, 256, False, (256, 320)), (6656, 5024, 256, False, (256, 320)), (6656, 5024, 320, True, (256, 320)),
    (2336, 11792, 256, False, (256, 256)), (2208, 5504, 256, False, (256, 224)), (2592, 9504, 256, False, (256, 224)),
    (1936, 11664, 256, False, (256, 192)), (3872, 12704, 320, False, (256, 160))])
def test_every_tile(M, N, K, per_row, takes):
    assert tile(M, N, K, per_row) == takes
    xb, wb = synth.normal_with_outliers(M, K, 1.0, 7400 + K, frac=0.01), synth.normal(N, K, 0.02, 7500 + N)
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
    y16 = torch.full((M, N + 16), 7.0, dtype=torch.bfloat16, device="cuda")
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_BF16, out=y16[:, :N], workspace=ws)
    assert torch.equal(y16, buf.to(torch.bfloat16))
    acc = buf[:, :N].clone()
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_F32_ACCUMULATE, out=acc, workspace=ws)
    assert torch.equal(acc, buf[:, :N] + buf[:, :N])
