"""GPU parity of the two-pass GEMM in each of its tiles, ragged at both edges, one tile per workgroup and several as one stream, against
the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import TWO_PASS, plan
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


def tile(M, N, K, per_row):
    route, shape = plan(M, N, K, workspace=True, row_scales=int(per_row))[:2]
    assert route == TWO_PASS
    return shape


@pytest.mark.parametrize("M,N,K,per_row,takes", [
    (1424, 13776, 320, False, (320, 320)), (3360, 12128, 256, False, (320, 320)), (2096, 19184, 320, False, (320, 320)),
    (1456, 10960, 320, False, (256, 320)), (6160, 5808, 256, False, (256, 320)), (2320, 14752, 320, True, (256, 320)),
    (1808, 15536, 256, False, (256, 256)), (3088, 3904, 320, False, (256, 224)), (2592, 9504, 256, False, (256, 224)),
    (1664, 13584, 320, False, (256, 192)), (3872, 12704, 320, False, (256, 160)),
    # two stages of K (a workgroup per tile), and four, the shortest that run as one stream: all that is loaded ahead is the next tile's
    (11328, 3216, 64, False, (256, 320)), (12848, 2848, 64, True, (256, 320)), (13888, 3216, 64, False, (320, 320)),
    (12816, 1568, 128, False, (256, 320)), (5520, 5904, 128, False, (256, 320)), (6304, 5184, 128, True, (256, 320)),
    (8464, 2832, 128, False, (320, 320)), (5424, 7648, 128, False, (320, 320))])
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


@pytest.mark.parametrize("M,N,K,per_row,splits", [(2896, 8096, 1024, False, 2), (2896, 8096, 1024, True, 2), (2592, 18240, 2112, False, 4),
                                                  (5088, 4032, 2048, True, 4), (3376, 9248, 4096, False, 8), (3376, 9248, 4096, True, 8)])
def test_split_last_round(M, N, K, per_row, splits):
    """256 x 256 tiles whose last round is split along K: against the kernel that a call without scratch takes, which sums in another order."""
    assert plan(M, N, K, workspace=True, row_scales=int(per_row))[1::2] == ((256, 256), splits) and plan(M, N, K)[0] != TWO_PASS
    xb, wb = synth.normal_with_outliers(M, K, 1.0, 7600 + K, frac=0.01), synth.normal(N, K, 0.02, 7700 + N)
    qx = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if per_row else 0))
    qw = nv.nvfp4_quantize(to_dev(wb), nv.LAYOUT_ROW)
    ws = torch.empty(nv.gemm_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, out=buf[:, :N], workspace=ws)
    ref = nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD).double()
    assert torch.all(buf[:, N:] == 7.0)
    # two FP32 sums of K / 32 steps each: sqrt(K / 32) 2^-24 of the result twice, 1.4e-6 at the most
    assert (buf[:, :N].double() - ref).norm() <= 3e-6 * ref.norm()
    assert torch.equal(nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_BF16, workspace=ws), buf[:, :N].to(torch.bfloat16))
    acc = buf[:, :N].clone()
    nv.nvfp4_gemm(qx, qw, nv.OP_DGRAD, nv.OUT_F32_ACCUMULATE, out=acc, workspace=ws)
    assert torch.equal(acc, buf[:, :N] + buf[:, :N])
