"""GPU parity of each tile shape of the GEMM straight from the packed codes, ragged in M and N: K shorter than a window of 128 or 256, a rest
of one to all wavefronts' turns behind whole windows, whole windows only, more windows than wavefronts."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import DIRECT, OWN_TILES, plan
from test_gpu_parity import GEMM_TOL, check_quantize, to_dev

pytestmark = pytest.mark.gpu


def shape(M, N, K):
    """(16-row blocks, 16-column blocks, wavefronts that split K, steps of 128 k to a window) that the product takes."""
    route, kind = plan(M, N, K)[:2]
    assert route == DIRECT
    out = (ctypes.c_int * 4)()
    i64 = ctypes.c_int64
    nv.load_library().nvfp4_internal_direct_shape(i64(M), i64(N), i64(K), int(kind == OWN_TILES), out)
    return tuple(out)


@pytest.mark.parametrize("M,N,K,takes", [
    (16, 16, 48, (1, 2, 4, 1)), (16, 16, 1616, (1, 2, 4, 2)), (16, 16, 1552, (1, 2, 8, 1)), (80, 8208, 144, (1, 2, 4, 1)), (4112, 16, 1216, (2, 2, 8, 1)), (2896, 80, 544, (2, 4, 8, 1)),
    (4112, 80, 16, (4, 3, 4, 1)), (1840, 272, 656, (4, 3, 4, 1)), (48, 8384, 1632, (4, 3, 4, 2)), (592, 2080, 768, (4, 3, 4, 2)),
    (208, 3248, 672, (4, 4, 4, 1)), (160, 4112, 128, (4, 4, 4, 1)), (176, 5568, 544, (4, 5, 4, 2)), (80, 8288, 1568, (4, 5, 4, 2)),
    (112, 8384, 768, (4, 5, 4, 2)), (144, 7936, 1552, (5, 5, 4, 2)), (208, 6784, 768, (5, 5, 4, 2)), (560, 3968, 560, (8, 5, 4, 2)),
    (2336, 976, 1360, (8, 5, 4, 2)), (1360, 1664, 1024, (8, 5, 4, 2)), (144, 8240, 144, (4, 4, 1, 1)), (528, 6560, 528, (6, 4, 1, 2)),
    (3664, 1184, 512, (6, 4, 1, 2)), (944, 8288, 544, (8, 5, 1, 2)), (1040, 7968, 512, (8, 5, 1, 2))])
def test_direct_shapes(M, N, K, takes):
    assert shape(M, N, K) == takes
    xb = synth.normal_with_outliers(M, K, 1.0, 7500 + M + K, frac=0.01)
    wb = synth.normal(K, N, 0.02, 7600 + N)
    qw, rw = check_quantize(wb, nv.LAYOUT_COL, nv.BLOCK_1x16)
    qx = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW)
    ref = oracle.gemm_f64(oracle.quantize(xb, oracle.ROW), rw["col"])
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")      # what lies beyond a row's N columns stays as it was
    nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, out=buf[:, :N])
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    assert np.abs(got[:, :N] - ref).max() <= 1e-4 * np.sqrt((ref * ref).mean())      # a wrong block is off by about that mean itself
    assert torch.equal(nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, nv.OUT_BF16), buf[:, :N].to(torch.bfloat16))
