"""GPU parity of the MXFP4 GEMM's narrower tiles (K a multiple of 512), ragged at both edges and with workgroups that run
several tiles as one stream, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


# 128, 160, 224 and 256 columns per tile: one tile each side of ragged; 512 / 460 tiles on 256 CUs; whole 256 x 256 tiles
@pytest.mark.parametrize("M,N,K", [(288, 160, 512), (1056, 1056, 1536), (4064, 5088, 512), (2016, 5088, 1536), (5088, 5088, 512),
                                   (4096, 4096, 1024)])
def test_mx_gemm_widths(M, N, K):
    ab, bb = synth.normal_with_outliers(M, K, 1.0, 930 + K, frac=0.01), synth.normal(N, K, 0.05, 931 + N)
    qa = nv.nvfp4_quantize(to_dev(ab), nv.LAYOUT_ROW, nv.BLOCK_MX32)
    qb = nv.nvfp4_quantize(to_dev(bb), nv.LAYOUT_ROW, nv.BLOCK_MX32)
    ref = oracle.mx_gemm_f64(oracle.mx_quantize(ab, oracle.ROW), oracle.mx_quantize(bb, oracle.ROW))
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_F32, out=buf[:, :N])
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)                 # nothing stored past a row's last column
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    d16 = nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_BF16)
    assert torch.equal(d16, buf[:, :N].to(torch.bfloat16))
    acc = buf[:, :N].clone()
    nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_F32_ACCUMULATE, out=acc)
    assert torch.equal(acc, buf[:, :N] + buf[:, :N])
