"""GPU parity of the quantizer at the edges of its workgroup tiles (cast pass 128 rows x 256 columns, amax pass 64 rows x 512
columns or more rows of a narrower tensor) and where an amax workgroup takes several pieces, bit for bit against the oracle: tensors of more than 176
tiles for these kernels; smaller ones, here too, have others."""
import ctypes

import pytest
import torch

import oracle
from paper_2509_25149_amd import binding as nv, synth
from test_gpu_parity import check_quantize, to_dev

pytestmark = pytest.mark.gpu

RC = nv.LAYOUT_ROW | nv.LAYOUT_COL


def kernels(rows, cols, layout=RC, rotated=False, block2d=False):
    """(cast pass of small tensors, amax pass of small tensors, reverse 1 and bands 2, sets of workgroups, log2 of the amax pass's lanes across)"""
    out, i64 = (ctypes.c_int * 5)(), ctypes.c_int64
    nv.load_library().nvfp4_internal_quantize_plan(i64(rows), i64(cols), layout & nv.LAYOUT_ROW, layout & nv.LAYOUT_COL, int(rotated), int(block2d), out)
    return tuple(out)


# inside one tile; exactly one; a 16-row and a 16-column remainder of a second; several tiles, odd scale rows (unaligned
# scale pieces); tensors so narrow that 2, 8 or 32 lanes of a wavefront span them in the amax pass, with a remainder of its row groups;
# more pieces of its work than workgroups, with few and with many column blocks (272 of them, 530).  The first group the same in tensors of more than 176 tiles:
# one row of tiles, inside it and exactly; a remainder each way; so many that both copies share a set of workgroups; 2, 8 and 32 lanes across
SMALL = [(112, 240), (128, 256), (144, 272), (656, 784), (2064, 48), (4112, 176)]
LARGE = [(112, 45296), (128, 45312), (144, 22800), (2064, 4112), (32784, 16), (22576, 48), (22672, 176), (144, 139024), (32, 271120)]


@pytest.mark.parametrize("rows,cols", SMALL + LARGE)
@pytest.mark.parametrize("mode", ["activation", "weight", "gradient", "row_only"])
def test_tile_edges(rows, cols, mode):
    rotated = mode in ("activation", "gradient")
    small, amax_small, _, sets, lane_bits = kernels(rows, cols, nv.LAYOUT_ROW if mode == "row_only" else RC, rotated, mode == "weight")
    one_piece = (rows, cols) in [(112, 240), (128, 256)]      # of amax_kernel, which then keeps them unless they are rotated
    assert small == ((rows, cols) in SMALL and mode != "weight")
    assert amax_small == ((rows, cols) in SMALL and cols >= 128 and (rotated or not one_piece))
    assert sets == (2 if rotated and -(-rows // 128) * -(-cols // 256) <= 256 else 1)
    assert lane_bits == {16: 1, 48: 3, 176: 5, 240: 5, 256: 5}.get(cols, 6)
    xb = synth.student_t3(rows, cols, 1e-3, rows + cols) if mode == "gradient" else \
        synth.normal_with_outliers(rows, cols, 1.0, rows + cols, frac=0.01)
    xb[-16:, -16:] = 0                                   # an all-zero 16x16 tile: stored scale 0
    xb[-1, 0] = 0x5000                                   # the tensor's largest magnitude in its last row
    if rows * cols > 1 << 22:
        xb[-1, 0], xb[rows // 2, -17] = 0x3f80, 0x5000   # in a column block and a row group that come late
    if mode == "activation":
        check_quantize(xb, RC, rht=True, rht_seed=11)
    elif mode == "weight":
        check_quantize(xb, RC, nv.BLOCK_16x16)
    elif mode == "gradient":
        check_quantize(xb, RC, rounding=nv.ROUND_SR, rht=True, rht_seed=12, sr_seed=13)
    else:
        check_quantize(xb, nv.LAYOUT_ROW)


# a row copy alone whose rows do not start on 128-byte lines: tiles dealt out in bands, one per XCD, with a remainder of the 8 and without
@pytest.mark.parametrize("rows,cols", [(2064, 2832), (2048, 2832), (11536, 528)])
def test_row_copy_in_bands(rows, cols):
    assert kernels(rows, cols, nv.LAYOUT_ROW)[:3] == (0, 0, 2)
    check_quantize(synth.normal_with_outliers(rows, cols, 1.0, 8100 + rows, frac=0.01), nv.LAYOUT_ROW)


@pytest.mark.parametrize("cols,ld,mode", [
    (16400, 16448, dict(layout_mask=RC, block_dim=nv.BLOCK_16x16)),          # rows on 128-byte lines by their padding: streamed
    (16400, 16400, dict(layout_mask=RC, rht_on_col=2, rht_seed=21)),         # rows anywhere, 269 MB: from the end
    (19504, 19504, dict(layout_mask=RC, rht_on_col=4, rht_seed=22)),         # 320 MB: streamed
    (19504, 19504, dict(layout_mask=nv.LAYOUT_ROW)),                         # the row copy alone, streamed and in bands
    (16400, 16400, dict(layout_mask=nv.LAYOUT_ROW)),                         # from the end and in bands
], ids=["16x16_padded", "d2", "d4", "row", "row_from_the_end"])
def test_beyond_the_memory_side_cache(cols, ld, mode):
    """Tensors of more than 256 MB: 144 rows repeated 57 times, so that the oracle's bytes for those repeat as well (same maximum, same
    blocks; nothing is drawn).  With the amax given, too: there the codes of rows that start anywhere leave by ordinary stores."""
    base, reps = 144, 57
    xb = synth.normal_with_outliers(base, cols, 1.0, 8200 + cols, frac=0.01)
    big = torch.zeros((base * reps, ld), dtype=torch.bfloat16, device="cuda")
    x = big[:, :cols]
    x.copy_(to_dev(xb).repeat(reps, 1))
    q = nv.nvfp4_quantize(x, **mode)
    given = nv.nvfp4_quantize_with_amax(x, nv.nvfp4_amax(x, mode.get("rht_on_col", 0), mode.get("rht_seed", 0)), **mode)
    ob = mode.get("block_dim", nv.BLOCK_1x16)
    ob = oracle.BLOCK_16x16 if ob == nv.BLOCK_16x16 else oracle.BLOCK_1x16
    for t in (q, given):
        r = oracle.quantize(xb, oracle.ROW, ob)
        assert torch.equal(t.row_codes.view(reps, base, -1), torch.from_numpy(r.codes).cuda().expand(reps, -1, -1))
        assert torch.equal(t.row_scales.view(reps, base, -1), torch.from_numpy(r.scales).cuda().expand(reps, -1, -1))
        assert t.row_ts.cpu().numpy()[1] == r.amax
        if mode["layout_mask"] & nv.LAYOUT_COL:
            d = mode.get("rht_on_col", 0)
            c = oracle.quantize(xb, oracle.COL, ob, oracle.RNE, d > 0, mode.get("rht_seed", 0), rht_dim=d or 16)
            assert torch.equal(t.col_codes.view(cols, reps, -1), torch.from_numpy(c.codes).cuda().unsqueeze(1).expand(-1, reps, -1))
            assert torch.equal(t.col_scales.view(cols, reps, -1), torch.from_numpy(c.scales).cuda().unsqueeze(1).expand(-1, reps, -1))
            assert t.col_ts.cpu().numpy()[1] == c.amax
