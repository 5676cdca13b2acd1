"""GPU parity of the GEMM straight from the packed codes (few tokens, small layers, K not a multiple of 64): each of its
tile shapes, and the 128 x 128 kernel of short contractions, at ragged edges of M, N and K, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import DIRECT, OWN_TILES, TILE_128, plan
from test_gpu_parity import GEMM_TOL, check_quantize, to_dev

pytestmark = pytest.mark.gpu


# tile shape the dispatch takes for it: 16x32 tiles (8 wavefronts; 4 for many tiles), 32x32, 64x48, 64x64 with K split among the
# wavefronts; 128x128 with a tile per wavefront; the 128x128 kernel.
# K: shorter than a step of 128; a step and a rest of one 16-block; whole steps; more steps than wavefronts, with a rest (every
# wavefront stages, reads back and stages again, and the sums of all of them are added).  The last seven: many rounds of tiles.
@pytest.mark.parametrize("M,N,K,kernel", [
    (16, 16, 16, (DIRECT, 0)), (48, 80, 112, (DIRECT, 0)), (16, 16400, 272, (DIRECT, 0)), (32, 5136, 400, (DIRECT, 0)), (32, 5136, 528, (DIRECT, 1)),
    (64, 9232, 128, (DIRECT, 2)), (80, 8208, 144, (DIRECT, 0)), (144, 5200, 1040, (DIRECT, 3)), (32, 5136, 2192, (DIRECT, 1)),
    (64, 9232, 1168, (DIRECT, 2)), (16, 16400, 1040, (DIRECT, 0)), (528, 5136, 1104, (DIRECT, OWN_TILES)), (272, 5136, 1104, (DIRECT, 3)),
    (2064, 8208, 16, (TILE_128, 0)), (2064, 4112, 80, (TILE_128, 0)), (1040, 8208, 208, (DIRECT, OWN_TILES)), (1040, 8208, 176, (TILE_128, 0)),
    (2064, 8208, 528, (DIRECT, OWN_TILES)), (4112, 4112, 528, (DIRECT, OWN_TILES)), (2064, 2064, 128, (DIRECT, OWN_TILES))])
@pytest.mark.parametrize("per_row", [False, True], ids=["tensor_scale", "row_scales"])
def test_direct_gemm(M, N, K, kernel, per_row):
    assert plan(M, N, K)[:2] == kernel
    xb = synth.normal_with_outliers(M, K, 1.0, 7000 + M + K, frac=0.01)
    wb = synth.normal(K, N, 0.02, 7100 + N)
    qw, rw = check_quantize(wb, nv.LAYOUT_COL, nv.BLOCK_16x16)
    qx = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if per_row else 0))
    rx = oracle.quantize_row_scales(xb, oracle.ROW) if per_row else oracle.quantize(xb, oracle.ROW)
    ref = oracle.gemm_f64(rx, rw["col"])
    ld = N + 16                      # what lies beyond a row's N columns stays as it was
    buf = torch.full((M, ld), 7.0, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, out=buf[:, :N])
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    ws = torch.empty(nv.gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    y16 = nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, nv.OUT_BF16, workspace=ws)          # bf16: the same sums, rounded once
    assert torch.equal(y16, buf[:, :N].to(torch.bfloat16))
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, nv.OUT_F32_ACCUMULATE, out=acc)
    assert torch.equal(acc, buf[:, :N] + 0.5)
