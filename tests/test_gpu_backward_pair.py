"""A small layer's Dgrad and Wgrad in one launch: bit for bit the two products on their own, for each pair of tile shapes that share a launch, both output
types of dX, dW overwritten and accumulated; and in a replayed HIP graph."""
import ctypes

import pytest
import torch

from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import to_dev

pytestmark = pytest.mark.gpu
RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


def operands(t, d_in, d_out):
    x, w, dy = (to_dev(b) for b in (synth.normal_with_outliers(t, d_in, 1.0, 5, frac=0.01), synth.normal(d_in, d_out, 0.02, 6), synth.student_t3(t, d_out, 1e-3, 7)))
    qx = nv.nvfp4_quantize(x, RC, rht_on_col=True, rht_seed=11)
    qw = nv.nvfp4_quantize(w, RC, nv.BLOCK_16x16)
    ws = torch.empty(max(nv.linear_workspace_bytes(t, d_in, d_out), 256), dtype=torch.uint8, device="cuda")
    i64 = ctypes.c_int64
    assert nv.load_library().nvfp4_internal_backward_pairs(i64(t), i64(d_in), i64(d_out), ctypes.c_size_t(ws.numel()))
    return qx, qw, dy, ws


# Dgrad's tiles + Wgrad's: 64 x 48 (K split) with itself, with 64 x 64 to each wavefront, with 64 x 64 (K split); the latter two with each of the three
SIZES = [(128, 4352, 256), (112, 4864, 464), (1040, 2064, 1296), (192, 2896, 256), (528, 4352, 272), (576, 5008, 400), (704, 3584, 256), (192, 4176, 256),
         (192, 4608, 464), (256, 3584, 256)]


@pytest.mark.parametrize("t,d_in,d_out", SIZES)
def test_one_launch_gives_the_bits_of_two(t, d_in, d_out):
    qx, qw, dy, ws = operands(t, d_in, d_out)
    start = torch.randn((d_in, d_out), device="cuda")
    for dtype in (nv.OUT_BF16, nv.OUT_F32):
        for accumulate in (False, True):
            dw = start.clone()
            dx, qdy = nv.nvfp4_linear_backward(dy, qx, qw, dw, ws, accumulate, 3, dtype)
            assert torch.equal(dx, nv.nvfp4_gemm(qdy, qw, nv.OP_DGRAD, dtype, workspace=ws))
            ref = start.clone()
            nv.nvfp4_gemm(qx, qdy, nv.OP_WGRAD, nv.OUT_F32_ACCUMULATE if accumulate else nv.OUT_F32, out=ref, workspace=ws)
            assert torch.equal(dw, ref)


def test_one_launch_replays_from_a_graph():
    t, d_in, d_out = 1040, 2064, 1296
    qx, qw, dy, ws = operands(t, d_in, d_out)
    dw, dx, qdy = torch.zeros((d_in, d_out), device="cuda"), torch.empty((t, d_in), dtype=torch.bfloat16, device="cuda"), nv.alloc_qtensor(t, d_out, RC)
    run = lambda: nv.nvfp4_linear_backward(dy, qx, qw, dw, ws, False, 3, qdy=qdy, dx=dx)
    run()
    torch.cuda.synchronize()
    want = dx.clone(), dw.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        dx.zero_()
        dw.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dx, want[0]) and torch.equal(dw, want[1])


def test_results_over_each_other_or_over_the_weights_codes():
    """The order of the calls holds where buffers are shared: dW, computed last, over dX; dW over the codes of W that Dgrad reads."""
    t, d_in, d_out = 1040, 2064, 1296
    qx, qw, dy, ws = operands(t, d_in, d_out)
    dw = torch.empty((d_in, d_out), device="cuda")
    dx, _ = nv.nvfp4_linear_backward(dy, qx, qw, dw, ws, False, 3)
    shared = torch.zeros((d_in, d_out), device="cuda")
    over = shared.view(-1).view(torch.bfloat16)[:t * d_in].view(t, d_in)
    nv.nvfp4_linear_backward(dy, qx, qw, shared, ws, False, 3, dx=over)
    assert torch.equal(shared, dw)
    codes = shared.view(-1).view(torch.uint8)[:qw.row_codes.numel()]
    codes.copy_(qw.row_codes.view(-1))
    qw.desc.row_codes = codes.data_ptr()
    dx2, _ = nv.nvfp4_linear_backward(dy, qx, qw, shared, ws, False, 3)
    assert torch.equal(dx2, dx) and torch.equal(shared, dw)
