"""GPU parity of the MXFP4 GEMM's tiles (K a multiple of 512), ragged at both edges and with workgroups that run
several tiles as one stream, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import mx_columns
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


# one tile each side of ragged; 256 tiles, 460 on 256 CUs; whole 256 x 256 tiles
@pytest.mark.parametrize("M,N,K,columns", [(288, 160, 512, 128), (1056, 1056, 1536, 128), (4064, 5088, 512, 320), (2016, 5088, 1536, 160), (5088, 5088, 512, 224),
                                           (4096, 4096, 1024, 256)])
def test_mx_gemm_widths(M, N, K, columns):
    assert mx_columns(M, N) == columns
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
