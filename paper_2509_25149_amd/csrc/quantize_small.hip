// The two passes of the NVFP4 quantizer (App. B Eq. 1-4; Sec. 4.2, 4.4; App. C) for tensors that fill the chip only with less work per lane than
// a 16-row x 8-column patch: 1x16 blocks, rotation sizes 2, 4, 16 or none.
//
// Such a call takes as long as the chain of one lane: load - rotate - maximum; launch; load - scale - encode - store.  A whole patch of eight
// columns is some 1300 instructions on a SIMD that has nothing else to do, so here a lane has
//   row copy   2 rows x 8 columns: a block is two neighbouring lanes, a row of a wavefront 32 lanes;
//   col copy   16 rows x 2 columns: the butterfly and both blocks in its registers; 64 lanes span 128 columns, a workgroup 64 rows;
//   amax pass  like the col copy,
// and each copy has workgroups of its own (the tensor, which the caches hold, is then read twice).  Random draws: a Philox call serves 8
// columns of a row, four lanes of the col copy: each of the four makes the calls of every fourth row and they trade words.
// us per call, patches of eight columns / here: 256 x 512 10.5 / 6.8, with stochastic rounding 12.7 / 7.7; 1040 x 1296 12.5 / 8.6, 14.6 / 9.7; row copy alone
// 64 x 5120 8.1 / 5.9.
#include "nvfp4_internal.h"
#include "quantize_tile.h"

namespace nvfp4 {
namespace {

constexpr int kRowTileRows = 16, kRowTileCols = 256;   // 8 x 32 lanes
constexpr int kColTileRows = 64, kColTileCols = 128;   // 4 wavefronts x 64 lanes

// Number `id` of n workgroups (dealt out to the 8 XCDs in turn) -> a numbering of which each XCD has a contiguous part.  The tiles leave pieces of 4 to 32 bytes
// (scales; codes of the col copy) of lines that neighbours fill up: row tiles are numbered along the rows, col tiles down the columns, so that the pieces meet in one
// L2.  us per call: X 1040 x 2064 9.9 -> 9.2, 2048 x 2816 12.5 -> 11.7, dY 1040 x 1296 8.7 -> 8.3.
__device__ __forceinline__ uint32_t xcd_contiguous(uint32_t id, uint32_t n) { return id < (n & ~7u) ? (id & 7) * (n >> 3) + (id >> 3) : id; }

// The 16 values of the lane's two columns, sign diagonal applied.
__device__ __forceinline__ void load_two_columns(const uint16_t* __restrict__ x, int64_t ld, int64_t row0, int64_t col0, uint32_t w[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) w[r] = *reinterpret_cast<const uint32_t*>(x + (row0 + r) * ld + col0);
}
__device__ __forceinline__ void signed_columns(const uint32_t w[16], uint32_t sign_mask, float lo[16], float hi[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t s = w[r] ^ (((sign_mask >> r) & 1u) * 0x80008000u);
    lo[r] = bf16_lo(s);
    hi[r] = bf16_hi(s);
  }
}

// Pass 1; what it leaves in the workspace is what amax_kernel leaves there (quantize.hip).
template <int kRht>
__global__ __launch_bounds__(kThreads) void amax_small_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols, int64_t ld, uint32_t sign_mask,
                                                              uint32_t col_blocks, uint32_t pieces, uint32_t* __restrict__ ws) {
  __shared__ uint32_t red[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t m_raw = 0, m_rot = 0;
  float f_rot = 0.0f;
#pragma unroll 1
  for (uint32_t piece = blockIdx.x; piece < pieces; piece += gridDim.x) {
    const uint32_t down = piece / col_blocks, across = piece - down * col_blocks;
    const int64_t row0 = static_cast<int64_t>(down) * kColTileRows + wave * 16, col0 = static_cast<int64_t>(across) * kColTileCols + lane * 2;
    if (col0 < cols && row0 < rows) {
      uint32_t w[16];
      load_two_columns(x, ld, row0, col0, w);
      uint32_t lo_max = 0, hi_max = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        lo_max = max(lo_max, w[r] & 0x7FFFu);
        hi_max = max(hi_max, w[r] & 0x7FFF0000u);
      }
      m_raw = max(m_raw, max(lo_max << 16, hi_max));
      if (kRht) {
        float lo[16], hi[16];
        signed_columns(w, sign_mask, lo, hi);
        butterfly_rows<kRht>(lo);
        butterfly_rows<kRht>(hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) f_rot = fmaxf(fmaxf(f_rot, fabsf(lo[r])), fabsf(hi[r]));
      }
    }
  }
  m_raw = wave_max_u32(m_raw);
  if (kRht) m_rot = wave_max_u32(__float_as_uint(rht_norm<kRht>() * f_rot));   // (once, on the maximum: rounding is monotone)
  if (lane == 0) {
    red[0][wave] = m_raw;
    red[1][wave] = m_rot;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t raw = max(max(red[0][0], red[0][1]), max(red[0][2], red[0][3]));
    uint32_t rot = max(max(red[1][0], red[1][1]), max(red[1][2], red[1][3]));
    if (raw >= 0x7F800000u) rot = max(rot, raw);
    ws[kWsHeader + blockIdx.x] = raw;
    ws[kWsHeader + gridDim.x + blockIdx.x] = rot;
  }
}

// Folds n per-workgroup maxima and fills the table of block encode scales 1 / (fp32(code) * s_dec) (App. B.2); every thread returns with the
// amax and Eq. 1's scales of the copy.
__device__ __forceinline__ void fold_and_tabulate(const uint32_t* __restrict__ maxima, uint32_t n, uint32_t (&red)[4], float (&lut)[128], float& amax,
                                                  float& s_enc, float& s_dec) {
  const int tid = threadIdx.x;
  uint32_t m = 0;
  for (uint32_t i = tid; i < n; i += kThreads) m = max(m, maxima[i]);
  m = wave_max_u32_lane63(m);
  if ((tid & 63) == 63) red[tid >> 6] = m;
  __syncthreads();
  amax = __uint_as_float(max(max(red[0], red[1]), max(red[2], red[3])));
  tensor_scales(amax, s_enc, s_dec);
  if (tid < 128) {
    const float den = e4m3_decode(tid) * s_dec;
    lut[tid] = (den == 0.0f || tid == 127) ? 0.0f : 1.0f / den;
  }
  __syncthreads();
}

template <bool kRow, bool kCol, int kRht, bool kSR>
__global__ __launch_bounds__(kThreads) void cast_small_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t cols, int64_t ld, const uint32_t* __restrict__ maxima, uint32_t n_maxima, uint32_t sign_mask,
    uint32_t key0, uint32_t key1, uint8_t* __restrict__ row_codes, uint8_t* __restrict__ row_scales, float* __restrict__ row_ts,
    uint8_t* __restrict__ col_codes, uint8_t* __restrict__ col_scales, float* __restrict__ col_ts, uint32_t row_wgs) {
  __shared__ __attribute__((aligned(16))) uint8_t st_codes[kCol ? 4 * kColTileCols * 8 : 16];                // [wavefront][column] x 8 bytes
  __shared__ __attribute__((aligned(16))) uint8_t st_scales[kCol ? 4 * kColTileCols : kRowTileRows * 16];    // [wavefront][column] or [row][16 blocks]
  __shared__ float lut[128];
  __shared__ uint32_t red[4];
  const int tid = threadIdx.x;
  float amax, s_enc, s_dec;

  if (kRow && (!kCol || blockIdx.x < row_wgs)) {
    const uint32_t wg = xcd_contiguous(blockIdx.x, kCol ? row_wgs : gridDim.x);
    const uint32_t across = static_cast<uint32_t>((cols + kRowTileCols - 1) / kRowTileCols), by = wg / across, bx = wg - by * across;
    const int l = tid & 31, row_in = (tid >> 5) * 2;
    const int64_t colblk = static_cast<int64_t>(bx) * kRowTileCols, col0 = colblk + l * 8, rowblk = static_cast<int64_t>(by) * kRowTileRows;
    const bool active = col0 < cols;   // rows come in multiples of 16
    uint4 raw[2] = {};
    if (active) {
#pragma unroll
      for (int r = 0; r < 2; ++r) raw[r] = *reinterpret_cast<const uint4*>(x + (rowblk + row_in + r) * ld + col0);
    }
    fold_and_tabulate(maxima, n_maxima, red, lut, amax, s_enc, s_dec);
    if (wg == 0 && tid == 0) {
      row_ts[0] = s_dec;
      row_ts[1] = amax;
    }
    if (active) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = patch_elem(raw[r], c);
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) m = fmaxf(m, fabsf(v[c]));
        m = fmaxf(m, lane_xor1(m));
        const uint32_t code = e4m3_encode(div_by_6(m) * s_enc);   // Eq. 2-3
        const float s_enc_b = lut[code];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] *= s_enc_b;              // Eq. 4
        uint32_t rnd[4] = {0, 0, 0, 0};
        if (kSR) philox4x32_10(static_cast<uint32_t>(col0 >> 3), static_cast<uint32_t>(rowblk + row_in + r), 0u, 0u, key0, key1, rnd);
        *reinterpret_cast<uint32_t*>(row_codes + (rowblk + row_in + r) * (cols / 2) + col0 / 2) = encode8<kSR>(v, rnd);
        if ((l & 1) == 0) st_scales[(row_in + r) * 16 + (l >> 1)] = static_cast<uint8_t>(code);
      }
    }
    __syncthreads();
    const int nblk = static_cast<int>(min<int64_t>(kRowTileCols, cols - colblk) / 16);
    const int64_t scale_ld = cols / 16;
    uint8_t* const dst = row_scales + rowblk * scale_ld + colblk / 16;
    if (nblk == 16 && (scale_ld & 15) == 0) {
      if (tid < kRowTileRows) *reinterpret_cast<uint4*>(dst + tid * scale_ld) = *reinterpret_cast<const uint4*>(st_scales + tid * 16);
    } else {
      const int r = tid >> 4, b = tid & 15;
      if (b < nblk) dst[r * scale_ld + b] = st_scales[r * 16 + b];
    }
    return;
  }

  if (kCol) {
    constexpr int kDiv = kRhtDiv<kRht>;
    const uint32_t wg = kRow ? xcd_contiguous(blockIdx.x - row_wgs, gridDim.x - row_wgs) : xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t down = static_cast<uint32_t>((rows + kColTileRows - 1) / kColTileRows), bx = wg / down, by = wg - bx * down;
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t colblk = static_cast<int64_t>(bx) * kColTileCols, col0 = colblk + lane * 2;
    const int64_t rowblk = static_cast<int64_t>(by) * kColTileRows, row0 = rowblk + wave * 16;
    const bool active = col0 < cols && row0 < rows;   // columns come in multiples of 16: a quad is in or out as a whole
    uint32_t w[16] = {};
    if (active) load_two_columns(x, ld, row0, col0, w);
    fold_and_tabulate(maxima + (kRht ? n_maxima : 0), n_maxima, red, lut, amax, s_enc, s_dec);
    if (wg == 0 && tid == 0) {
      col_ts[0] = s_dec;
      col_ts[1] = amax;
    }
    // the lane's word of each row's draws: low half for its first column, high half for its second
    uint32_t draws[16] = {};
    if (kSR) {
      const int mine = lane & 3;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint32_t rnd[4];   // of row 4 g + mine
        philox4x32_10(static_cast<uint32_t>(col0 >> 3), static_cast<uint32_t>(row0 + 4 * g + mine), 0u, 0u, key0, key1, rnd);
        // row 4 g + k: lane k of the quad has it; every lane takes the word of its own number
#define NVFP4_TAKE(K)                                                                                                          \
  {                                                                                                                             \
    uint32_t t[4];                                                                                                              \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) t[i] = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(rnd[i]), (K) * 0x55, 0xF, 0xF, true)); \
    draws[4 * g + (K)] = mine == 0 ? t[0] : mine == 1 ? t[1] : mine == 2 ? t[2] : t[3];                                        \
  }
        NVFP4_TAKE(0) NVFP4_TAKE(1) NVFP4_TAKE(2) NVFP4_TAKE(3)
#undef NVFP4_TAKE
      }
    }
    if (active) {
      float v[2][16];
      signed_columns(w, sign_mask, v[0], v[1]);
      uint2 out[2];
      uint32_t code[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        butterfly_rows<kRht>(v[c]);
        normalise<kRht>(v[c]);
        float m = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) m = fmaxf(fmaxf(m, fabsf(v[c][r])), fabsf(v[c][r + 1]));
        if (kDiv != 1) m *= 1.0f / kDiv;
        code[c] = e4m3_encode(div_by_6(m) * s_enc);
        const float s_enc_b = lut[code[c]];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[c][r] *= s_enc_b;
        uint32_t half[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (!kSR) {
            const uint32_t none[4] = {0, 0, 0, 0};
            half[h] = encode8<false, kDiv>(v[c] + 8 * h, none);
          } else {
            const float* u = v[c] + 8 * h;
            auto d = [&](int t) { return c ? draws[8 * h + t] & 0xFFFF0000u : draws[8 * h + t] << 16; };
            uint32_t e = any_word(u[0]), o = any_word(u[1]);
            cvt_sr_single_into<0, kDiv>(e, u[0], d(0));
            cvt_sr_single_into<1, kDiv>(e, u[2], d(2));
            cvt_sr_single_into<2, kDiv>(e, u[4], d(4));
            cvt_sr_single_into<3, kDiv>(e, u[6], d(6));
            cvt_sr_single_into<0, kDiv>(o, u[1], d(1));
            cvt_sr_single_into<1, kDiv>(o, u[3], d(3));
            cvt_sr_single_into<2, kDiv>(o, u[5], d(5));
            cvt_sr_single_into<3, kDiv>(o, u[7], d(7));
            half[h] = interleave_nibbles(e, o);
          }
        }
        out[c] = make_uint2(half[0], half[1]);
      }
      *reinterpret_cast<uint4*>(st_codes + (wave * kColTileCols + lane * 2) * 8) = make_uint4(out[0].x, out[0].y, out[1].x, out[1].y);
      *reinterpret_cast<uint16_t*>(st_scales + wave * kColTileCols + lane * 2) = static_cast<uint16_t>(code[0] | code[1] << 8);
    }
    __syncthreads();
    const int tile_cols = static_cast<int>(min<int64_t>(kColTileCols, cols - colblk)), tile_groups = static_cast<int>(min<int64_t>(kColTileRows, rows - rowblk) / 16);
    const int64_t code_ld = rows / 2, scale_ld = rows / 16;
    const int j = tid >> 1, pair = tid & 1;   // pieces of 16 bytes: column j, two 16-row groups
    if (j < tile_cols) {
      const uint2 a = *reinterpret_cast<const uint2*>(st_codes + (2 * pair * kColTileCols + j) * 8);
      const uint2 b = *reinterpret_cast<const uint2*>(st_codes + ((2 * pair + 1) * kColTileCols + j) * 8);
      uint8_t* dst = col_codes + (colblk + j) * code_ld + rowblk / 2 + pair * 16;
      if ((code_ld & 15) == 0 && 2 * pair + 1 < tile_groups) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(a.x, a.y, b.x, b.y);
      } else {
        if (2 * pair < tile_groups) *reinterpret_cast<uint2*>(dst) = a;
        if (2 * pair + 1 < tile_groups) *reinterpret_cast<uint2*>(dst + 8) = b;
      }
    }
    if (tid < tile_cols) {   // one column: up to 4 scale bytes
      uint8_t sc[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) sc[g] = st_scales[g * kColTileCols + tid];
      uint8_t* dst = col_scales + (colblk + tid) * scale_ld + rowblk / 16;
      if (tile_groups == 4 && (scale_ld & 3) == 0) {
        *reinterpret_cast<uint32_t*>(dst) = sc[0] | (sc[1] << 8) | (sc[2] << 16) | (static_cast<uint32_t>(sc[3]) << 24);
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (g < tile_groups) dst[g] = sc[g];
      }
    }
  }
}

uint32_t tiles(int64_t n, int64_t of) { return static_cast<uint32_t>((n + of - 1) / of); }

}  // namespace

// Workgroups of the amax pass: pieces of 64 rows x 128 columns, at most 256 of them at a time.  (Two words each fit the workspace whatever the
// shape, which has 2 (rows + cols) and at least one piece's share for each 64 rows and 128 columns.)
uint32_t small_amax_workgroups(const QuantizeArgs& a) {
  const uint32_t pieces = tiles(a.rows, kColTileRows) * tiles(a.cols, kColTileCols);
  return pieces < 256 ? pieces : 256;
}

template <int kRht>
void launch_amax_small(const QuantizeArgs& a, hipStream_t s) {
  const uint32_t col_blocks = tiles(a.cols, kColTileCols), pieces = col_blocks * tiles(a.rows, kColTileRows);
  hipLaunchKernelGGL(amax_small_kernel<kRht>, dim3(small_amax_workgroups(a)), dim3(kThreads), 0, s, static_cast<const uint16_t*>(a.x), a.rows, a.cols, a.ld,
                     a.sign_mask, col_blocks, pieces, a.ws);
}

template <bool kRow, bool kCol, int kRht>
void launch_cast_small(const QuantizeArgs& a, const uint32_t* maxima, uint32_t n_maxima, hipStream_t s) {
  const uint32_t row_wgs = kRow ? tiles(a.rows, kRowTileRows) * tiles(a.cols, kRowTileCols) : 0;
  const uint32_t col_wgs = kCol ? tiles(a.rows, kColTileRows) * tiles(a.cols, kColTileCols) : 0;
  const auto kernel = a.sr ? &cast_small_kernel<kRow, kCol, kRht, true> : &cast_small_kernel<kRow, kCol, kRht, false>;
  hipLaunchKernelGGL(kernel, dim3(row_wgs + col_wgs), dim3(kThreads), 0, s, static_cast<const uint16_t*>(a.x), a.rows, a.cols, a.ld, maxima, n_maxima,
                     a.sign_mask, a.key0, a.key1, a.row_codes, a.row_scales, a.row_ts, a.col_codes, a.col_scales, a.col_ts, row_wgs);
}

template void launch_amax_small<0>(const QuantizeArgs&, hipStream_t);
template void launch_amax_small<2>(const QuantizeArgs&, hipStream_t);
template void launch_amax_small<4>(const QuantizeArgs&, hipStream_t);
template void launch_amax_small<16>(const QuantizeArgs&, hipStream_t);
template void launch_cast_small<true, true, 0>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<true, false, 0>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<false, true, 0>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<true, true, 2>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<false, true, 2>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<true, true, 4>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<false, true, 4>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<true, true, 16>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);
template void launch_cast_small<false, true, 16>(const QuantizeArgs&, const uint32_t*, uint32_t, hipStream_t);

}  // namespace nvfp4
