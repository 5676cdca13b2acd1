// NVFP4 quantizer kernels for gfx950 (App. B Eq. 1-4; Sec. 4.2-4.4; App. C).
//
// Work decomposition shared by both passes: a lane owns a 16-row x 8-column
// patch of the bf16 tensor (sixteen 128-bit loads, one per row).  In the amax
// pass a wavefront spans 16 rows x 512 columns (more rows of a narrower tensor) at a time; in the
// cast pass it is one patch per lane, two 16-row groups x 256 columns, and a
// 256-thread workgroup covers 128 rows x 256 columns.  With this patch
//   - a 1x16 block of the row copy is split over two neighbouring lanes
//     (one cross-lane exchange of the half-block amax),
//   - a 1x16 block of the col copy (16 consecutive rows of one column) sits
//     entirely in one lane's registers, so the Hadamard butterfly and the
//     block amax need no cross-lane traffic,
//   - a 16x16 weight tile is exactly two neighbouring lanes,
//   - the eight columns of one row are the eight elements served by one
//     Philox call, whose output is shared by the row and the col copy.
// Row codes leave as one dword per lane and row (128 contiguous bytes per
// 16-row group).  The transposed col copy, its scales and the row scales are staged
// in LDS and written back as contiguous 128-bit / 64-bit pieces: 64 bytes of
// codes per column per workgroup instead of scattered 8-byte stores.
#include "nvfp4_internal.h"
#include "quantize_tile.h"

namespace nvfp4 {


// ---------------------------------------------------------------- pass 1: amax (App. B.1)
// Every workgroup writes its own maxima (raw tensor / rotated tensor) into its
// slot of the workspace; whoever needs the tensor's folds the slots.  No atomics:
// thousands of same-address atomics serialise in L2 and cost more than the pass.
// The raw maximum is always taken, also when only a rotated copy is asked for: it is the one place where a NaN in
// the input shows (the floating-point maxima of the rotated values skip NaNs), and a non-finite one is carried over into
// the rotated maximum -- here, not where the maxima are folded: there the two words may be a caller's, who gives each for itself.
// A piece of work is 4 wavefronts x 64 lanes; `lanes` = 1 << lane_bits of a wavefront (64, fewer for a tensor narrower than 512
// columns) span the columns of one 16-row group.  Pieces are numbered column by column, then down the rows, and dealt to the
// workgroups in turn, so that a tensor of any proportions keeps every one of them and every lane at work.  (With whole column
// blocks to a workgroup 1024 x 133120 took 57 us, 1048576 x 16 208.)
template <int kRht>   // kRht: 0, or the rotation size 2, 4 or 16 (sign_mask: the d signs repeated over 16 bits)
__global__ __launch_bounds__(kThreads) void amax_kernel(const uint16_t* __restrict__ x, int64_t rows,
                                                        int64_t cols, int64_t ld, uint32_t sign_mask, int lane_bits, uint32_t col_blocks,
                                                        uint32_t pieces, uint32_t* __restrict__ ws) {
  __shared__ uint32_t red[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, groups_per_wave = 64 >> lane_bits;
  const int64_t ngroups = rows / 16;
  uint32_t m_raw = 0, m_rot = 0;
  float f_rot = 0.0f;
#pragma unroll 1
  for (uint32_t piece = blockIdx.x; piece < pieces; piece += gridDim.x) {
    const uint32_t down = piece / col_blocks, across = piece - down * col_blocks;
    const int64_t group = (static_cast<int64_t>(down) * 4 + wave) * groups_per_wave + (lane >> lane_bits);
    const int64_t col0 = (static_cast<int64_t>(across) << (lane_bits + 3)) + (lane & ((1 << lane_bits) - 1)) * 8;
    if (col0 < cols && group < ngroups) {
      Patch p;
      load_patch(x, ld, group * 16, col0, p);
      m_raw = max(m_raw, patch_amax_bits(p));
      if (kRht) {
        // The normalisation is applied once to the maximum: rounding is monotone, so
        // max_i fl(c v_i) = fl(c max_i v_i).
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float lo[16], hi[16];
          signed_column_pair(p, t, sign_mask, lo, hi);
          butterfly_rows<kRht>(lo);
          butterfly_rows<kRht>(hi);
#pragma unroll
          for (int r = 0; r < 16; ++r) f_rot = fmaxf(fmaxf(f_rot, fabsf(lo[r])), fabsf(hi[r]));
        }
      }
    }
  }
  m_raw = wave_max_u32(m_raw);
  if (kRht) m_rot = wave_max_u32(__float_as_uint(rht_norm<kRht>() * f_rot));
  if (lane == 0) {
    red[0][wave] = m_raw;
    red[1][wave] = m_rot;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t nwg = gridDim.x, wg = blockIdx.x;
    const uint32_t raw = max(max(red[0][0], red[0][1]), max(red[0][2], red[0][3]));
    uint32_t rot = max(max(red[1][0], red[1][1]), max(red[1][2], red[1][3]));
    if (raw >= 0x7F800000u) rot = max(rot, raw);
    ws[kWsHeader + wg] = raw;
    ws[kWsHeader + nwg + wg] = rot;
  }
}

// ---------------------------------------------------------------- pass 2: cast
// A workgroup is four wavefronts with one patch per lane: a wavefront spans two 16-row groups x 256 columns, a workgroup 128
// rows x 256 columns, which is 64 bytes of codes per column of the col copy and 128 per row of the row copy.  (One
// patch per lane instead of two 16-row groups one after the other: 256 x 512 22.7 -> 13.1 us per call, 1040 x 2064 49 -> 15.7.
// Wavefronts of 16 rows x 512 columns leave 32-byte pieces of col codes, 8192 x 5120 47 -> 57 us; 64 x 128 no better than this.)
// A 4- or 16-point rotation's normalisation is left to the conversions, whose scale operand divides by a power of two: 128 multiplications of a patch's 2050 (3100 with
// stochastic rounding) instructions less; X 8192 x 5120 45.9 -> 45.1 us, dY 8192 x 20480 SR 188.6 -> 185.4.
// What bounds it: large tensors the memory system (all calls, both passes, bytes over time: W 5120 x 20480 6.2 TB/s where a
// plain copy of this card runs at 4.6 - 5.1), with stochastic rounding the vector pipe (Philox and one conversion per
// value), small ones the chain load - amax - scale - table - codes of one patch.
// maxima: n raw maxima, then n rotated ones (pass 1's slots; n = 1: the tensor's own), folded by every workgroup while its
// patch is on its way from memory -- a launch of its own for that cost 5 us and two gaps between kernels.
// Codes leave with non-temporal stores: nothing reads them in this call, and in the memory-side cache they push out the tensor
// that pass 1 has left there (W 104 -> 86 us, dY 8192 x 20480 SR 223 -> 213, X 8192 x 5120 47.8 -> 46.8).
// (After a pass 1, that is; for calls with the amax given see cast_memory.)
enum CastMemory { kCachedLoads = 0, kStreamedLoads = 1, kStreamedLoadsCachedStores = 2 };
template <int kMemory>
using CastTile = Staged<8, 32, kMemory != kStreamedLoadsCachedStores>;
enum { kWalkReverse = 1, kWalkBands = 2, kWalkStrips = 4 };   // see cast_walk
__device__ __forceinline__ float to_scalar(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }

// kMemory: see cast_memory (a template argument because a branch around the patch's loads makes every one of them wait at
// its end: dY 8192 x 20480 SR 232 us).
template <bool kRow, bool kCol, int kRht, bool kSR, bool k2D, int kMemory>   // kRht as in amax_kernel
// With stochastic rounding the draws of a patch (64 registers beside its own 64) left room for two wavefronts per SIMD, which did
// not cover each other's loads and stores; columns one at a time instead of in pairs bring both copies under 168 registers (with
// eight parked in LDS), i.e. to three: dY 8192 x 20480 209 -> 189 us, 8192 x 5120 61 -> 57.
__global__ __launch_bounds__(kThreads, kSR && kRow && kCol && !k2D ? 3 : 2) void cast_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t cols, int64_t ld,
    const uint32_t* __restrict__ maxima, uint32_t n_maxima, uint32_t sign_mask, uint32_t key0, uint32_t key1,
    uint8_t* __restrict__ row_codes, uint8_t* __restrict__ row_scales, float* __restrict__ row_ts,
    uint8_t* __restrict__ col_codes, uint8_t* __restrict__ col_scales, float* __restrict__ col_ts, int walk) {
  using T = CastTile<kMemory>;
  __shared__ __attribute__((aligned(16))) uint8_t st_col_codes[kCol ? T::kColCodesBytes : 16];
  __shared__ __attribute__((aligned(16))) uint8_t st_col_scales[kCol ? T::kColScalesBytes : 16];
  __shared__ __attribute__((aligned(16))) uint8_t st_row_scales[kRow ? T::kRowScalesBytes : 16];
  __shared__ float lut_row[128], lut_col[128];  // block encode scale per stored E4M3 code
  __shared__ uint32_t red[2][4];
  __shared__ __attribute__((aligned(16))) uint4 stash[kSR && kRow && kCol ? 2 * kThreads : 1];

  const int tid = threadIdx.x, lane = tid & (T::kLanes - 1), wave = tid >> 6;
  const int gl = tid / T::kLanes;                // group index inside the tile
  unsigned bx = blockIdx.x, by = blockIdx.y;
  if (walk & (kWalkBands | kWalkStrips)) {
    const unsigned id = by * gridDim.x + bx, band = gridDim.x * gridDim.y >> 3;
    const unsigned to = id < band * 8 ? (id & 7) * band + (id >> 3) : id;
    if (walk & kWalkStrips) {
      const unsigned strip = to / (8 * gridDim.y), in = to - strip * (8 * gridDim.y), width = min(8u, gridDim.x - strip * 8);
      by = width == 8 ? in >> 3 : in / width;
      bx = strip * 8 + in - by * width;
    } else {
      by = to / gridDim.x;
      bx = to - by * gridDim.x;
    }
  }
  if (walk & kWalkReverse) {
    bx = gridDim.x - 1 - bx;
    by = gridDim.y - 1 - by;
  }
  const int64_t colblk = static_cast<int64_t>(bx) * T::kCols;
  const int64_t col0 = colblk + lane * 8;
  const int64_t group0 = static_cast<int64_t>(by) * T::kGroups, ngroups = rows / 16;
  const int64_t group = group0 + gl, row0 = group * 16;
  const bool active = col0 < cols && group < ngroups;
  // A small tensor's two copies are made by two sets of workgroups (see launch_cast).
  const bool do_row = kRow && (gridDim.z == 1 || blockIdx.z == 0), do_col = kCol && (gridDim.z == 1 || blockIdx.z == 1);

  Patch p;
  if (active) load_patch<kMemory != kCachedLoads>(x, ld, row0, col0, p);

  uint32_t m_raw = 0, m_rot = 0;
  for (uint32_t i = tid; i < n_maxima; i += kThreads) {
    m_raw = max(m_raw, maxima[i]);
    if (kRht) m_rot = max(m_rot, maxima[n_maxima + i]);
  }
  m_raw = wave_max_u32_lane63(m_raw);
  if (kRht) m_rot = wave_max_u32_lane63(m_rot);
  if ((tid & 63) == 63) {
    red[0][wave] = m_raw;
    red[1][wave] = m_rot;
  }
  __syncthreads();
  m_raw = max(max(red[0][0], red[0][1]), max(red[0][2], red[0][3]));
  m_rot = max(max(red[1][0], red[1][1]), max(red[1][2], red[1][3]));

  // App. B.1 Eq. 1, from the amax of pass 1.
  const float amax_raw = __uint_as_float(m_raw);
  const float amax_col = kRht ? __uint_as_float(m_rot) : amax_raw;
  float s_enc_r, s_dec_r, s_enc_c, s_dec_c;
  tensor_scales(amax_raw, s_enc_r, s_dec_r);
  tensor_scales(amax_col, s_enc_c, s_dec_c);
  s_enc_r = to_scalar(s_enc_r);   // the same in every lane: no vector register for them
  s_enc_c = to_scalar(s_enc_c);
  if (bx == 0 && by == 0 && tid == 0) {
    if (do_row) { row_ts[0] = s_dec_r; row_ts[1] = amax_raw; }
    if (do_col) { col_ts[0] = s_dec_c; col_ts[1] = amax_col; }
  }
  // "real" block encode scale 1 / (fp32(code) * s_dec) for each of the 127 codes (App. B.2)
  {
    const int code = tid & 127;
    const float den = e4m3_decode(code) * (tid < 128 ? s_dec_r : s_dec_c);
    const float inv = (den == 0.0f || code == 127) ? 0.0f : 1.0f / den;
    if (tid < 128) lut_row[code] = inv; else lut_col[code] = inv;
  }
  __syncthreads();

  if (active) {
    // Random words: one Philox call per row serves the row's 8 columns.
    uint32_t rnd[16][4];
    if (kSR) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        philox4x32_10(static_cast<uint32_t>(col0 >> 3), static_cast<uint32_t>(row0 + r), 0u, 0u, key0, key1, rnd[r]);
    }

    // 16x16 tile amax (Sec. 4.3): this lane's 16x8 half and the neighbour's.
    float s_enc_tile = 0.0f;
    uint32_t tile_code = 0;
    if (k2D) {
      uint32_t m = patch_amax_bits(p);
      m = max(m, lane_xor1(m));
      tile_code = e4m3_encode(div_by_6(__uint_as_float(m)) * s_enc_r);   // Eq. 2-3
      s_enc_tile = lut_row[tile_code];
    }

    if (do_row)
      row_pass<kSR, k2D, T>(p, rnd, lane, gl, s_enc_r, lut_row, s_enc_tile, tile_code, row_codes + row0 * (cols / 2) + col0 / 2,
                            cols / 2, st_row_scales);

    if (do_col) {
      if (kSR) {
        // one column at a time, in order: with the draws in registers there is no room for two, and eight of the words that
        // hold columns 6 and 7 wait in LDS meanwhile (the assembly statement keeps the compiler from remembering them)
        if (kRow) {
          stash[tid] = make_uint4(p.raw[0].w, p.raw[1].w, p.raw[2].w, p.raw[3].w);
          stash[kThreads + tid] = make_uint4(p.raw[4].w, p.raw[5].w, p.raw[6].w, p.raw[7].w);
          asm volatile("" ::"v"(stash + tid) : "memory");
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (kRow && c == 6) {
            const uint4 a = stash[tid], b = stash[kThreads + tid];
            p.raw[0].w = a.x, p.raw[1].w = a.y, p.raw[2].w = a.z, p.raw[3].w = a.w;
            p.raw[4].w = b.x, p.raw[5].w = b.y, p.raw[6].w = b.z, p.raw[7].w = b.w;
          }
          float v[16];
          signed_column(p, c, sign_mask, v);
          butterfly_rows<kRht>(v);
          normalise<kRht>(v);
          emit_column<kSR, k2D, T, kRhtDiv<kRht>>(v, c, rnd, lane, gl, s_enc_c, lut_col, s_enc_tile, tile_code, st_col_codes, st_col_scales);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float lo[16], hi[16];
          // Without a rotation sign_mask is 0 at run time; it is still applied, so that these values are not
          // recognised as the row pass's: keeping all 128 of those alive costs more registers than there are.
          signed_column_pair(p, t, sign_mask, lo, hi);
          butterfly_rows<kRht>(lo);
          butterfly_rows<kRht>(hi);
          normalise<kRht>(lo);
          normalise<kRht>(hi);
          emit_column<kSR, k2D, T, kRhtDiv<kRht>>(lo, 2 * t, rnd, lane, gl, s_enc_c, lut_col, s_enc_tile, tile_code, st_col_codes, st_col_scales);
          emit_column<kSR, k2D, T, kRhtDiv<kRht>>(hi, 2 * t + 1, rnd, lane, gl, s_enc_c, lut_col, s_enc_tile, tile_code, st_col_codes, st_col_scales);
        }
      }
    }
  }
  __syncthreads();

  write_back_tile<kRow, kCol, kThreads, T>(tid, rows, cols, group0, ngroups, colblk, st_col_codes, st_col_scales,
                                           st_row_scales, row_scales, col_codes, col_scales, do_row, do_col);
}

// ---------------------------------------------------------------- host side

size_t quantize_workspace_bytes(int64_t rows, int64_t cols) {
  const int64_t gx = (cols + kWaveCols - 1) / kWaveCols, gy = (rows / 16 + kGroupsPerBlock - 1) / kGroupsPerBlock;
  // raw, col-rotated, row-rotated maxima per workgroup; or, with one scale per row of each copy, amax and encode scale
  // per row and per column
  const size_t per_tensor = static_cast<size_t>(kWsHeader + 3 * gx * gy), per_row = quantize_rowscale_workspace_words(rows, cols);
  return (per_tensor > per_row ? per_tensor : per_row) * sizeof(uint32_t);
}

// How the cast pass goes over memory.  After pass 1, which has just streamed the tensor front to back through the 256 MB
// memory-side cache:
//   above 128 MB from its end (what comes last is what the cache still holds; a smaller tensor it holds whole);
//   above 256 MB, where most of it is gone again, from the front and with non-temporal loads, which leave the tail alone until the
//   walk gets there (dY 8192 x 20480, 335 MB: RNE 173 -> 154 us, SR 212 -> 203; at 251 MB they are the slower: 145 against 153).  Where rows
//   do not start on 128-byte lines, two workgroups fetch each border line and the cache has to hold it between them: there from
//   304 MB on (8208 x 16400, 269 MB: X 185 us streamed, 178 from the end; 8176 x 19472, 318 MB: 222 / 223).
// With the amax given: non-temporal loads above 256 MB, and where rows do not start on 128-byte lines ordinary stores of the codes --
// nothing of the tensor is to be kept in the cache, and it puts the pieces of border lines together (15552 x 13648 259 -> 178 us, 8176 x
// 20464 149 either way; on 128-byte lines it depends on the shape: 8192 x 20480 126 -> 107, 4096 x 76800 213 -> 231).
// The row copy alone, rows not on 128-byte lines: neighbouring tiles, which share those lines and the border lines of the codes, go to
// workgroups of one XCD (they are dealt out round robin), an eighth of the grid to each: 5104 x 20464 91 -> 80 us, 8176 x 5104 38.8 -> 35.1,
// 1920 x 31504 56 -> 50.  With both copies it loses above 200 MB (5104 x 20464 129 -> 137), with few rows too (272 x 131088 36 -> 37).
// The others in strips of 8 tiles across, walked downwards, an eighth of the sequence to each XCD: a tile leaves 16 bytes of a row's scales, 8 bytes of a column's and
// 64 of its codes, which fill lines of 128 together with neighbours to the side and below; from workgroups all over the chip each L2 has its part of such a line and writes it
// by itself (without the scales W took 6 us less, with them as non-temporal stores 9 to 30 more).  W 5120 x 20480 85.8 -> 82.8 us, 5136 x 20496 125 -> 117, X 4096 x 5120
// 28.5 -> 27.7, dY 8208 x 16400 186 -> 180, the row copy alone 8192 x 20480 122 -> 117; strips of 4 alike, of 16 84.4 for the first.
// Some aligned tensors along their rows all the same (along_rows_pays): the cache holds the last rows of a tensor somewhat larger than itself, and where the tiles across are a
// multiple of 8 (of 4, of 2) an XCD meets every (every second, every fourth) tile of a column that way too.  us, along the rows / in strips: both copies above 256 MB, X 8192 x 20480 150 / 159.
// One copy of a tensor whose amax is given, which has not just been read: the row copy above 256 MB (163 sizes: 1.09 times the time in strips; 9216 x 19968 86 / 97, 3840 x 65792 114 / 189), with
// stochastic rounding any (227: 0.99 if the tensor is in the cache, 1.035 if not; 4352 x 10496 48.4 / 50.4); the col copy up to 256 MB with a multiple of 4 tiles across (111: 1.014, 1.04; 13312 x
// 6144 47.6 / 51.1).  The col copy of 256 to 384 MB, taller than wide, with an even number of tiles across (118: 1.058; 79616 x 2048 119 / 143, 14080 x 12288 125 / 134) or stochastic
// rounding (76: 1.025; 39680 x 3840 138 / 144); an odd number of tiles 0.967 (19456 x 9984 166 / 155), wider than tall 0.94.
constexpr int64_t kCacheBytes = int64_t{256} << 20;
static bool lines_aligned(const QuantizeArgs& a) { return a.ld % 64 == 0 && reinterpret_cast<uintptr_t>(a.x) % 128 == 0; }
static CastMemory cast_memory(const QuantizeArgs& a) {
  const int64_t bytes = a.rows * a.cols * 2;
  if (lines_aligned(a)) return bytes > kCacheBytes ? kStreamedLoads : kCachedLoads;
  if (!a.do_amax) return bytes > kCacheBytes ? kStreamedLoadsCachedStores : kCachedLoads;
  return bytes > kCacheBytes / 16 * 19 ? kStreamedLoads : kCachedLoads;
}
// Of an aligned tensor.
static bool along_rows_pays(const QuantizeArgs& a) {
  using T = CastTile<kCachedLoads>;   // the tile is the same for all
  const int64_t bytes = a.rows * a.cols * 2, across = (a.cols + T::kCols - 1) / T::kCols;
  const bool large = bytes > kCacheBytes;
  if (a.want_row && a.want_col) return large;
  if (a.do_amax) return a.want_col && large && bytes <= kCacheBytes / 2 * 3 && a.rows > a.cols && (across % 2 == 0 || a.sr);
  return a.want_row ? large || a.sr : !large && across % 4 == 0;
}
static int cast_walk(const QuantizeArgs& a) {
  const bool reverse = a.do_amax && a.rows * a.cols * 2 > kCacheBytes / 2 && cast_memory(a) == kCachedLoads;
  const bool bands = !a.want_col && !lines_aligned(a) && a.rows >= 1024;
  const bool strips = !bands && !(lines_aligned(a) && along_rows_pays(a));
  return (reverse ? kWalkReverse : 0) | (bands ? kWalkBands : strips ? kWalkStrips : 0);
}

// Workgroups of the amax pass, at most 512: two to a CU keep enough loads in flight, and every workgroup of the cast pass
// folds their maxima (dY 8192 x 20480: 512 218 us per call, 1024 222, 2048 236).
// Two words each fit the workspace whatever the shape: it has 2 (rows + cols), and pieces of 64 rows x 512 columns, or of more
// rows of a narrower tensor, are fewer.
struct AmaxWork {
  int lane_bits;
  uint32_t col_blocks, pieces, workgroups;
};
static AmaxWork amax_work(const QuantizeArgs& a) {
  constexpr uint32_t kMaxAmaxWgs = 512;
  AmaxWork w{6, 0, 0, 0};
  while (w.lane_bits > 1 && a.cols <= (int64_t{4} << w.lane_bits)) --w.lane_bits;   // half the lanes span it
  const int64_t rows = int64_t{64} << (6 - w.lane_bits);                             // of a piece
  w.col_blocks = static_cast<uint32_t>((a.cols + (int64_t{8} << w.lane_bits) - 1) >> (w.lane_bits + 3));
  w.pieces = static_cast<uint32_t>(w.col_blocks * ((a.rows + rows - 1) / rows));
  w.workgroups = w.pieces < kMaxAmaxWgs ? w.pieces : kMaxAmaxWgs;
  return w;
}

// Up to 176 tiles of 128 x 256 the kernels with less work per lane (quantize_small.hip): a call takes as long as one lane's chain does.  us per call, this
// cast pass / those: X 256 x 512 10.5 / 6.8, X 2048 x 2048 (128 tiles) 11.5 / 9.8, X 4096 x 1040 (160) 13.7 / 12.8, X 2048 x 4096 (256) 14.1 / 16.4;
// stochastic rounding 12.7 / 7.7, 13.6 / 12.4, 17.2 / 16.2, 17.7 / 20.8; the row copy alone 64 x 5120 8.1 / 5.9, 2048 x 4096 10.6 / 11.0.
static int64_t cast_tiles(const QuantizeArgs& a) {
  using T = CastTile<kCachedLoads>;   // the tile is the same for all
  return ((a.cols + T::kCols - 1) / T::kCols) * ((a.rows / 16 + T::kGroups - 1) / T::kGroups);
}
static bool use_cast_small(const QuantizeArgs& a) { return cast_tiles(a) <= 176 && !a.block2d; }
// Its wavefronts span 128 columns.  What one workgroup of amax_kernel covers, unrotated, has no long chain and is left to it: a second workgroup costs more than
// the shorter loads gain (us, amax_kernel / amax_small_kernel: 64 x 256 3.7 / 3.9, a weight's call 7.5 / 7.9; 64 x 1024 4.1 / 3.9; rotated 64 x 256 4.9 / 4.2).
static bool use_amax_small(const QuantizeArgs& a) {
  const bool rotated = a.want_col && a.rht_dim != 0;
  return cast_tiles(a) <= 176 && a.cols >= 128 && (rotated || amax_work(a).pieces > 1);
}

// Up to 256 workgroups (one per CU) the call takes as long as one patch does: each copy gets workgroups of its own, though the
// patch is then read twice.  us, one set / two: X 2048 x 4096 (256 workgroups) 15.0 / 12.9, dY 4096 x 4096 (512) 28.4 / 31.8.  16x16 blocks have
// little work per patch: 2048 x 4096 10.3 / 10.8.
static unsigned cast_sets(const QuantizeArgs& a) { return a.want_row && a.want_col && !a.block2d && cast_tiles(a) <= 256 ? 2 : 1; }

template <bool kRow, bool kCol, int kRht, bool kSR, bool k2D>
static void launch_cast(const QuantizeArgs& a, const uint32_t* maxima, uint32_t n_maxima, hipStream_t s) {
  using T = CastTile<kCachedLoads>;   // the tile is the same for all
  const unsigned gx = static_cast<unsigned>((a.cols + T::kCols - 1) / T::kCols), gy = static_cast<unsigned>((a.rows / 16 + T::kGroups - 1) / T::kGroups);
  const dim3 grid(gx, gy, cast_sets(a));
  const CastMemory m = cast_memory(a);
  const auto kernel = m == kCachedLoads     ? &cast_kernel<kRow, kCol, kRht, kSR, k2D, kCachedLoads>
                      : m == kStreamedLoads ? &cast_kernel<kRow, kCol, kRht, kSR, k2D, kStreamedLoads>
                                            : &cast_kernel<kRow, kCol, kRht, kSR, k2D, kStreamedLoadsCachedStores>;
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s,
                     static_cast<const uint16_t*>(a.x), a.rows, a.cols, a.ld, maxima, n_maxima, a.sign_mask, a.key0,
                     a.key1, a.row_codes, a.row_scales, a.row_ts, a.col_codes, a.col_scales, a.col_ts, cast_walk(a));
}

template <bool kRow, bool kCol, int kRht>
static void launch_passes(const QuantizeArgs& a, hipStream_t s) {
  uint32_t n_maxima = 1;
  if (a.do_amax) {
    if (use_amax_small(a)) {
      n_maxima = small_amax_workgroups(a);
      launch_amax_small<kRht>(a, s);
    } else {
      const AmaxWork w = amax_work(a);
      n_maxima = w.workgroups;
      hipLaunchKernelGGL((amax_kernel<kRht>), dim3(w.workgroups), dim3(kThreads), 0, s, static_cast<const uint16_t*>(a.x), a.rows, a.cols,
                         a.ld, a.sign_mask, w.lane_bits, w.col_blocks, w.pieces, a.ws);
    }
    // the cast pass folds the maxima itself; only a caller of the amax alone needs them folded
    if (!a.do_cast) hipLaunchKernelGGL(amax_finalize_kernel, dim3(1), dim3(1024), 0, s, a.ws, n_maxima, a.amax_copy);
  }
  if (!a.do_cast) return;
  const uint32_t* maxima = a.do_amax ? a.ws + kWsHeader : a.ws;
  if (a.block2d) {
    if (a.sr) launch_cast<kRow, kCol, 0, true, true>(a, maxima, n_maxima, s);
    else launch_cast<kRow, kCol, 0, false, true>(a, maxima, n_maxima, s);
  } else if (use_cast_small(a)) {
    launch_cast_small<kRow, kCol, kRht>(a, maxima, n_maxima, s);
  } else {
    if (a.sr) launch_cast<kRow, kCol, kRht, true, false>(a, maxima, n_maxima, s);
    else launch_cast<kRow, kCol, kRht, false, false>(a, maxima, n_maxima, s);
  }
}

hipError_t launch_quantize(const QuantizeArgs& a, hipStream_t s) {
  const int rht = a.want_col ? a.rht_dim : 0;
  if (a.scale_per_row) return launch_quantize_rowscale(a, s);
  if (a.row_rht) return launch_quantize_rowrot(a, s);
  if (rht > 16) return launch_quantize_wide(a, s);
  if (rht == 16) {
    if (a.want_row) launch_passes<true, true, 16>(a, s); else launch_passes<false, true, 16>(a, s);
  } else if (rht == 4) {
    if (a.want_row) launch_passes<true, true, 4>(a, s); else launch_passes<false, true, 4>(a, s);
  } else if (rht == 2) {
    if (a.want_row) launch_passes<true, true, 2>(a, s); else launch_passes<false, true, 2>(a, s);
  } else {
    if (a.want_row && a.want_col) launch_passes<true, true, 0>(a, s);
    else if (a.want_row) launch_passes<true, false, 0>(a, s);
    else launch_passes<false, true, 0>(a, s);
  }
  return hipGetLastError();
}

}  // namespace nvfp4

// For the tests, not part of the ABI: which kernels nvfp4_quantize takes for a contiguous tensor of these sizes (rotation up to 16, one scale
// per tensor; rotated: the col copy is; options: 1 16x16 blocks, 2 stochastic rounding, 4 the amax given).  out: cast pass (0 cast_kernel, 1 cast_small_kernel), amax pass (likewise), cast_kernel's walk (kWalkReverse | kWalkBands | kWalkStrips), sets of its workgroups,
// log2 of amax_kernel's lanes across.
extern "C" void nvfp4_internal_quantize_plan(int64_t rows, int64_t cols, int want_row, int want_col, int rotated, int options, int* out) {
  using namespace nvfp4;
  QuantizeArgs a{};
  a.rows = rows;
  a.cols = a.ld = cols;
  a.want_row = want_row;
  a.want_col = want_col;
  a.block2d = options & 1;
  a.sr = options & 2;
  a.rht_dim = rotated ? 16 : 0;
  a.do_amax = !(options & 4);
  a.do_cast = true;
  out[0] = use_cast_small(a);
  out[1] = use_amax_small(a);
  out[2] = cast_walk(a);
  out[3] = static_cast<int>(cast_sets(a));
  out[4] = amax_work(a).lane_bits;
}
