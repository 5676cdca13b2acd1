"""Which kernel an NVFP4 product takes (host code only): the library's own plan, asked through the query that it exports for tests.
Here: each class of products takes the kernel that was measured to be the faster one for it."""
import ctypes
import os
import random

import pytest

from paper_2509_25149_amd import binding as nv

TWO_PASS, FUSED_256, TILE_128, DIRECT = range(4)
OWN_TILES = 4                        # the direct kernel's shape without a split of K


@pytest.fixture(scope="module", autouse=True)
def library():
    if not os.path.exists(nv.LIB_PATH):
        pytest.skip("libnvfp4_hip.so not built")


def plan(M, N, K, bf16=False, accumulate=False, workspace=0, decoded=0, row_scales=0):
    """(route, shape, tiles of a split last round, splits) as launched; shape: (rows, columns) of a two-pass tile, the direct kernel's kind of tile;
    workspace: bytes, or True for what the library asks for; decoded, row_scales: bit 0 A, bit 1 B."""
    out = (ctypes.c_int * 5)()
    if workspace is True:
        workspace = nv.gemm_workspace_bytes(M, N, K)
    i64 = ctypes.c_int64
    nv.load_library().nvfp4_internal_gemm_plan(i64(M), i64(N), i64(K), int(bf16), int(accumulate), ctypes.c_size_t(workspace), decoded, row_scales, out)
    return out[0], (out[1], out[2]) if out[0] == TWO_PASS else out[1], out[3], out[4]


def mx_columns(M, N):
    """Of an MXFP4 product's tile where K is a multiple of 512."""
    i64 = ctypes.c_int64
    return 32 * nv.load_library().nvfp4_internal_mx_gemm_width(i64(M), i64(N))


@pytest.mark.parametrize("M,N", [(2048, 2048), (2048, 8192), (5120, 20480), (4096, 5120), (8176, 1296)])
@pytest.mark.parametrize("K", [16, 48, 80, 144, 208, 272, 336, 400])
@pytest.mark.parametrize("bf16,accumulate", [(False, False), (True, False), (False, True)], ids=["f32", "bf16", "accumulate"])
def test_short_contractions_with_a_large_result_do_not_split_k(M, N, K, bf16, accumulate):
    """The result's bytes are the work: no wavefront may wait for others that have no step of K.  5120 x 20480 x 16 (FP32) took 193 us
    with K split over four wavefronts, 80 in 128 x 128 tiles."""
    for workspace in (0, True):
        route, shape = plan(M, N, K, bf16, accumulate, workspace)[:2]
        assert route == TILE_128 or (route, shape) == (DIRECT, OWN_TILES)
    if K <= 48 and M * N > 8e6:
        assert route == TILE_128


@pytest.mark.parametrize("M,N,K", [(5120, 20480, 1040), (5120, 20480, 2064), (4096, 5120, 1040), (8176, 1296, 1040), (8176, 20464, 5136)])
def test_large_products_of_a_ragged_contraction_keep_whole_tiles(M, N, K):
    assert plan(M, N, K)[:2] == (DIRECT, OWN_TILES)      # 5120 x 20480 x 1040: 314 us; 385 with K split, 369 in the 128 x 128 kernel


@pytest.mark.parametrize("M,N,K,shape", [(16, 20480, 5136, 0), (32, 5120, 5136, 1), (64, 20480, 5136, 2), (512, 5120, 5136, 3),
                                         (64, 20480, 5120, 2), (512, 5120, 5120, 3), (1040, 1296, 2064, 2), (256, 256, 512, 0)])
def test_few_tokens_and_small_layers_split_k(M, N, K, shape):
    for workspace in (0, True):
        assert plan(M, N, K, True, False, workspace)[:2] == (DIRECT, shape)


@pytest.mark.parametrize("M,N,K", [(768, 2128, 64), (2240, 816, 32), (1040, 1296, 16), (320, 5680, 64), (1024, 1024, 80)])
def test_small_results_split_k_while_all_workgroups_are_resident(M, N, K):
    """768 x 2128 x 64 accumulated: 8.0 us with K split, 10.9 in 128 x 128 tiles of four wavefronts' own; FP32 alike."""
    for accumulate in (False, True):
        for workspace in (0, True):
            route, shape = plan(M, N, K, False, accumulate, workspace)[:2]
            assert route == DIRECT and shape < OWN_TILES


@pytest.mark.parametrize("M,N,K,tile", [(8192, 20480, 5120, (256, 320)), (8192, 5120, 20480, (256, 320)), (5120, 20480, 8192, (320, 320)),
                                        (5120, 5120, 4096, (320, 320)), (2048, 5120, 5120, (256, 160)), (4096, 5120, 5120, (256, 320)),
                                        (960, 18016, 2560, (256, 320)), (2944, 8192, 1024, (256, 256))])
def test_large_products_take_the_two_pass_route(M, N, K, tile):
    assert plan(M, N, K, workspace=True)[:2] == (TWO_PASS, tile)
    assert plan(M, N, K, workspace=0)[0] in (FUSED_256, DIRECT)


@pytest.mark.parametrize("M,N,columns", [(8192, 20480, 320), (4096, 5120, 320), (5120, 5120, 224), (4096, 4096, 256), (2048, 5120, 160), (512, 5120, 128)])
def test_mxfp4_tile_widths(M, N, columns):
    assert mx_columns(M, N) == columns


# us in the direct kernel / two-pass, accumulated
@pytest.mark.parametrize("M,N,K,route", [(11648, 1328, 1152, DIRECT),      # 53 / 68
                                         (1344, 11248, 1280, DIRECT), (896, 17280, 8960, DIRECT),
                                         (864, 17504, 2496, TWO_PASS)])    # 1.13 to 1.26 times as fast as the direct kernel
def test_what_a_larger_tile_gains_counts_for_the_route_in_contractions_of_1536_to_4096(M, N, K, route):
    for accumulate in (False, True):
        assert plan(M, N, K, accumulate=accumulate, workspace=True)[0] == route


@pytest.mark.parametrize("M,N,columns", [(6656, 14240, 256), (9600, 9216, 256), (7328, 11712, 256),     # five rounds of 320 columns, six of 256: 186 / 166 us at K = 3584
                                         (13824, 12672, 320), (8160, 4992, 320), (4608, 4224, 320)])      # nine and ten; three of 224; two of 160
def test_mxfp4_widest_tile_has_to_promise_more_than_one_percent(M, N, columns):
    assert mx_columns(M, N) == columns


def test_accumulating_products_of_a_short_contraction_keep_a_wide_tile_unless_a_narrower_one_saves_rounds():
    """1620 tiles of 256 columns are 7 rounds, 2538 of 160 columns 10 of 0.68: 3 % less, not enough where the result is read too."""
    M, N, K = 13776, 7472, 512
    assert plan(M, N, K, accumulate=True, workspace=True)[:2] == (TWO_PASS, (256, 256))
    assert plan(M, N, K, workspace=True)[:2] == (TWO_PASS, (256, 160))


@pytest.mark.parametrize("K", [2 ** 27 + 16, 2 ** 29, 2 ** 31 + 16, 2 ** 33 + 64])
def test_contractions_beyond_the_direct_kernels_offsets_take_a_kernel_that_has_none(K):
    """The direct kernel's byte offsets within 16 rows are 32 bits wide (K <= 2^27); the other two count K in 64."""
    for M, N in ((16, 16), (16, 4096), (512, 512)):
        assert plan(M, N, K)[0] == (TILE_128 if K % 64 else FUSED_256)
    assert plan(16, 16, 2 ** 27)[0] == DIRECT


def test_results_too_large_for_one_launch_of_a_kernel_take_another():
    # tile rows of the 128 x 128 kernel are the launch's second dimension: 65535 of them at the most
    assert plan(65535 * 128, 128, 16)[0] == TILE_128
    assert plan(65535 * 128 + 16, 128, 16)[0] == DIRECT
    # 16 x 32 tiles: 256 threads each, under 2^32 in all
    assert plan(2 ** 26, 128, 16)[:2] != (DIRECT, 0)
    # 32-bit rows of the direct kernel
    assert plan(16, 2 ** 31, 16)[0] == TILE_128


def test_one_kernel_for_all_output_types():
    """bf16 results are the FP32 ones rounded, accumulated ones the FP32 ones added: to the last bit only if the same sums are taken in the
    same order.  (Two-pass tiles of any width take them in the same order unless the last round is split, which needs K >= 1024.)"""
    rng = random.Random(7)
    size = lambda lo, hi: max(16, int(lo * (hi / lo) ** rng.random()) // 16 * 16)
    for _ in range(4000):
        M, N, K = size(16, 20480), size(16, 20480), size(16, 20480)
        K = K if rng.random() < 0.5 else max(64, K // 64 * 64)
        for workspace, decoded in ((0, 0), (0, 3), (True, 0), (True, 2)):
            f32 = plan(M, N, K, False, False, workspace, decoded)
            assert plan(M, N, K, True, False, workspace, decoded) == f32
            accumulated = plan(M, N, K, False, True, workspace, decoded)
            assert accumulated == f32 or (f32[0] == accumulated[0] == TWO_PASS and f32[2:] == accumulated[2:] == (0, 1) and K < 1024)


def test_workspace_without_room_for_partial_tiles_still_serves_the_two_pass_route():
    M, N, K = 8256, 4096, 4096                                   # 528 tiles: the last 16 split 8 ways
    operands = (M + N) * K * 2
    assert plan(M, N, K, workspace=True) == (TWO_PASS, (256, 256), 16, 8)
    assert nv.gemm_workspace_bytes(M, N, K) == operands + 16 * 8 * 2 ** 18
    route, tile, tail, splits = plan(M, N, K, workspace=operands)
    assert (route, tail, splits) == (TWO_PASS, 0, 1) and tile != (256, 256)    # three whole rounds of 256 columns or fewer of other tiles
    assert plan(M, N, K, workspace=operands - 256)[0] != TWO_PASS
    # with both operands decoded nothing is needed; with room for the partial tiles alone the split is back
    assert plan(M, N, K, decoded=3) == (TWO_PASS, tile, 0, 1)
    assert plan(M, N, K, workspace=16 * 8 * 2 ** 18, decoded=3) == (TWO_PASS, (256, 256), 16, 8)
    assert plan(M, N, K, workspace=N * K * 2, decoded=1)[0] == TWO_PASS


@pytest.mark.parametrize("M,N,K", [(4352, 4096, 4096), (8192, 5120, 20480), (5120, 20480, 8192), (4096, 5120, 5120), (2048, 5120, 5120)])
def test_tiles_without_a_split_ask_for_no_room_for_partial_ones(M, N, K):
    """Their rounds of 256 x 256 tiles would be partial; they run in others."""
    operands = (M + N) * K * 2
    assert nv.gemm_workspace_bytes(M, N, K) == operands
    with_room = plan(M, N, K, workspace=operands + 2 ** 27)
    assert with_room[0] == TWO_PASS and with_room[1] != (256, 256) and with_room[2:] == (0, 1)
    assert plan(M, N, K, workspace=operands) == with_room
    assert plan(M, N, K, decoded=3) == plan(M, N, K, workspace=2 ** 27, decoded=3) == with_room


def test_the_workspace_query_covers_either_kind_of_scales():
    M, N, K = 5088, 4032, 2048                                   # 320 x 320 tiles, which a scale per row rules out
    assert plan(M, N, K, workspace=True) == (TWO_PASS, (320, 320), 0, 1)
    for row_scales in (1, 2, 3):
        assert plan(M, N, K, workspace=True, row_scales=row_scales) == (TWO_PASS, (256, 256), 64, 4)
    assert nv.gemm_workspace_bytes(M, N, K) == (M + N) * K * 2 + 64 * 4 * 2 ** 18


def test_what_the_query_asks_for_is_enough_and_no_more_than_is_used():
    """More room changes nothing, and where it asks for partial tiles one of the kinds of scales has them."""
    rng = random.Random(9)
    size = lambda: max(256, int(256 * 60 ** rng.random()) // 16 * 16)
    split = 0
    for _ in range(3000):
        M, N, K = size(), size(), size() // 64 * 64
        need = nv.gemm_workspace_bytes(M, N, K)
        plans = [plan(M, N, K, workspace=need, decoded=3, row_scales=r) for r in (0, 1, 2, 3)]
        assert plans == [plan(M, N, K, workspace=2 ** 42, decoded=3, row_scales=r) for r in (0, 1, 2, 3)]
        partials = need - ((M + N) * K * 2 + 255) // 256 * 256
        assert partials == max(p[2] * p[3] if p[3] > 1 else 0 for p in plans) * 2 ** 18
        split += partials > 0
    assert split > 20


def direct_shapes():
    """The direct kernel's tile shapes by number: (16-row blocks, 16-column blocks, wavefronts that split K, steps of 128 k to a window)."""
    out, shapes = (ctypes.c_int * 4)(), []
    while nv.load_library().nvfp4_internal_direct_shape_at(len(shapes), out):
        shapes.append(tuple(out))
    return shapes


def fits(shape, M, N, K):
    i64 = ctypes.c_int64
    return bool(nv.load_library().nvfp4_internal_direct_fits(i64(M), i64(N), i64(K), shape))


def test_what_a_direct_shape_can_do():
    shapes = direct_shapes()
    assert len(set(shapes)) == len(shapes) and {s[3] for s in shapes} == {1, 2}
    for i, (mb, nb, wk, steps) in enumerate(shapes):
        assert fits(i, 16, 16, 16) == fits(i, 4096, 4096, 240) == (steps == 1)       # less than a window of 256 k: windows of 128 only
        assert fits(i, 16, 16, 256) and fits(i, 16, 16, 2 ** 27) and not fits(i, 16, 16, 2 ** 27 + 16)
        assert not fits(i, 16, 2 ** 31, 256)
        own = 2 if wk == 1 else 1
        rows = 2 ** 32 // (wk * own * own * 64) * mb * own * 16                      # a column of tiles of 2^32 threads
        if rows < 2 ** 31:
            assert not fits(i, rows, 16, 256) and fits(i, rows - mb * own * 16, 16, 256)
    assert not fits(-1, 16, 16, 256) and not fits(len(shapes), 16, 16, 256)
