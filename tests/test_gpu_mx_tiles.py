"""GPU parity of the MXFP4 GEMM in each of its tile widths, ragged at both edges, one tile per workgroup and several as one stream, over
one, two and three chunks of scales, against the oracle's binary64 product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import mx_columns
from test_gpu_parity import GEMM_TOL, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,columns", [(96, 96, 512, 128), (1312, 5568, 512, 160), (4960, 3904, 1024, 160), (1824, 5184, 1536, 224), (4768, 4192, 512, 224),
                                           (3104, 4288, 512, 256), (5216, 5440, 1024, 256), (3104, 4960, 512, 320), (4896, 3136, 1536, 320),
                                           (5664, 5696, 1024, 320)])
def test_every_width(M, N, K, columns):
    assert mx_columns(M, N) == columns
    ab, bb = synth.normal_with_outliers(M, K, 1.0, 940 + K, frac=0.01), synth.normal(N, K, 0.05, 941 + N)
    qa = nv.nvfp4_quantize(to_dev(ab), nv.LAYOUT_ROW, nv.BLOCK_MX32)
    qb = nv.nvfp4_quantize(to_dev(bb), nv.LAYOUT_ROW, nv.BLOCK_MX32)
    ref = oracle.mx_gemm_f64(oracle.mx_quantize(ab, oracle.ROW), oracle.mx_quantize(bb, oracle.ROW))
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")
    nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_F32, out=buf[:, :N])
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)                 # nothing stored past a row's last column
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    d16 = torch.full((M, N + 16), 7.0, dtype=torch.bfloat16, device="cuda")
    nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_BF16, out=d16[:, :N])
    assert torch.equal(d16, buf.to(torch.bfloat16))
    acc = buf[:, :N].clone()
    nv.nvfp4_gemm(qa, qb, nv.OP_DGRAD, nv.OUT_F32_ACCUMULATE, out=acc)
    assert torch.equal(acc, buf[:, :N] + buf[:, :N])
