"""GPU parity of each tile shape of the GEMM straight from the packed codes, ragged in M and N: forced, over what a wavefront can have of K, with each kind
of result and of tensor scale; and through the library's own choice."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gemm_routes import DIRECT, direct_shapes, fits, plan
from test_gpu_parity import GEMM_TOL, check_quantize, to_dev

pytestmark = pytest.mark.gpu

NUM_SHAPES = 13      # test_every_shape_is_named


def force(shape, a, b, out, out_dtype):
    rc = nv.load_library().nvfp4_internal_gemm_direct(ctypes.byref(a.desc), ctypes.byref(b.desc), nv.OP_FPROP, ctypes.c_void_p(out.data_ptr()), out_dtype,
                                                      ctypes.c_int64(out.stride(0)), shape, ctypes.c_void_p(nv._stream()))
    if rc:
        raise nv.NVFP4Error(rc)
    return out


def windows_per_wavefront(K, wk, steps):
    """Whole windows and rest (k) of each of the wavefronts that split K: window i goes to wavefront i % wk, and so does the rest as if it were the next."""
    full = K // (128 * steps)
    return [(len(range(w, full, wk)), K - full * 128 * steps if full % wk == w else 0) for w in range(wk)]


def check_results(run, M, N, ref):
    """FP32 results within tolerance and nothing beyond them, bf16 and accumulated ones from the same sums."""
    buf = torch.full((M, N + 16), 7.0, dtype=torch.float32, device="cuda")      # what lies beyond a row's N columns stays as it was
    run(buf[:, :N], nv.OUT_F32)
    got = buf.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)
    assert np.linalg.norm(got[:, :N].astype(np.float64) - ref) <= GEMM_TOL * np.linalg.norm(ref)
    assert np.abs(got[:, :N] - ref).max() <= 1e-4 * np.sqrt((ref * ref).mean())      # a wrong block is off by about that mean itself
    assert torch.equal(run(torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), nv.OUT_BF16), buf[:, :N].to(torch.bfloat16))
    acc = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda")
    assert torch.equal(run(acc, nv.OUT_F32_ACCUMULATE), buf[:, :N] + 0.5)


def operands(M, N, K, per_row):
    xb = synth.normal_with_outliers(M, K, 1.0, 7500 + M + K, frac=0.01)
    wb = synth.normal(K, N, 0.02, 7600 + N)
    qw, rw = check_quantize(wb, nv.LAYOUT_COL, nv.BLOCK_1x16)
    qx = nv.nvfp4_quantize(to_dev(xb), nv.LAYOUT_ROW | (nv.LAYOUT_ROW_SCALES if per_row else 0))
    rx = oracle.quantize_row_scales(xb, oracle.ROW) if per_row else oracle.quantize(xb, oracle.ROW)
    return qx, qw, oracle.gemm_f64(rx, rw["col"])


def test_every_shape_is_named():
    assert len(direct_shapes()) == NUM_SHAPES


# What of K there is: less than a window of 128; one window; one and a rest, which is the next wavefront's; a window to each and the rest to the first; three windows
# to each (the loop's steady state: what it loads is multiplied two windows later) and none; five to the first, four to the others and a rest
KINDS = ("16", "112", "one", "one+16", "each+48", "three", "five+176")


@pytest.mark.parametrize("per_row", [False, True], ids=["tensor_scale", "row_scales"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", range(NUM_SHAPES))
def test_forced_shape(shape, kind, per_row):
    mb, nb, wk, steps = direct_shapes()[shape]
    w, own = 128 * steps, 2 if wk == 1 else 1
    K = {"16": 16, "112": 112, "one": w, "one+16": w + 16, "each+48": w * wk + 48, "three": 3 * w * wk, "five+176": (4 * wk + 1) * w + (176 if steps == 2 else 80)}[kind]
    parts = windows_per_wavefront(K, wk, steps)
    assert kind != "three" or parts == [(3, 0)] * wk
    assert kind != "five+176" or (parts[0][0] == 5 and parts[1 % wk] == (4 if wk > 1 else 5, 176 if steps == 2 else 80))
    M, N = mb * 16 * own + 16, nb * 16 * own + 48                               # two tiles each way, the second with one 16-row block or three columns
    assert fits(shape, M, N, K) == (K >= w or steps == 1)
    qx, qw, ref = operands(M, N, K, per_row)
    if not fits(shape, M, N, K):
        with pytest.raises(nv.NVFP4Error):
            force(shape, qx, qw, torch.empty((M, N), dtype=torch.float32, device="cuda"), nv.OUT_F32)
        return
    check_results(lambda out, kind: force(shape, qx, qw, out, kind), M, N, ref)


def test_unknown_shapes_are_refused():
    qx, qw, _ = operands(16, 16, 256, False)
    for shape in (-1, NUM_SHAPES):
        with pytest.raises(nv.NVFP4Error):
            force(shape, qx, qw, torch.empty((16, 16), dtype=torch.float32, device="cuda"), nv.OUT_F32)


@pytest.mark.parametrize("M,N,K", [
    (16, 16, 48), (16, 16, 1616), (16, 16, 1552), (80, 8208, 144), (4112, 16, 1216), (2896, 80, 544), (4112, 80, 16), (1840, 272, 656), (48, 8384, 1632),
    (592, 2080, 768), (208, 3248, 672), (160, 4112, 128), (176, 5568, 544), (80, 8288, 1568), (112, 8384, 768), (144, 7936, 1552), (208, 6784, 768),
    (560, 3968, 560), (2336, 976, 1360), (1360, 1664, 1024), (144, 8240, 144), (528, 6560, 528), (3664, 1184, 512), (944, 8288, 544), (1040, 7968, 512)])
def test_direct_products(M, N, K):
    assert plan(M, N, K)[0] == DIRECT
    qx, qw, ref = operands(M, N, K, False)
    def run(out, kind):
        return nv.nvfp4_gemm(qx, qw, nv.OP_FPROP, kind, out=out)
    check_results(run, M, N, ref)
