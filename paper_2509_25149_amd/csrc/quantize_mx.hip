// MXFP4 quantizer for gfx950: the paper's comparison format (Sec. 2: E2M1
// elements, blocks of 32, one UE8M0 power-of-two scale per block; App. B.4:
// the scale is amax_b / 6 rounded up to a power of two so nothing saturates;
// Sec. 5: a 32-point random Hadamard rotation on the Wgrad operands).
//
// There is no tensor-level scale, so one pass over the tensor is enough.
// Work decomposition: a lane owns 16 rows x 8 columns (sixteen 128-bit loads); a wavefront 32 rows x 256 columns,
// rows 0 - 15 in its lower half and 16 - 31 in its upper; a 256-thread workgroup 128 rows x 256 columns.  A row-copy
// block (32 columns of one row) is four neighbouring lanes (two cross-lane maxima).  A col-copy block (32 rows of one
// column) is a lane and its counterpart 32 lanes on: stages h = 1 .. 8 of the 32-point butterfly run in each, then
// v_permlane32_swap_b32 exchanges half of the values -- after it a lane holds both partners of eight pairs (i, i + 16), rows
// i = 0 - 7 and 16 - 23 in the lower half, 8 - 15 and 24 - 31 in the upper -- and stage 16 runs in each again.  Row codes leave as
// one dword per lane and row; everything else is staged in LDS and written back as
// contiguous pieces (64 bytes of codes per column per workgroup).  (Non-temporal stores of the codes made
// the calls by themselves faster -- X 8192 x 5120 47 -> 41 us -- but the GEMM behind them, which reads the codes as they are, slower by
// more: training step 4096 x 5120 x 5120 289 -> 302 us.)
// What bounds it: up to one round of workgroups the chain load - rotate - maximum - codes - store of one patch, beyond that memory (8192 x 20480
// 523 MB in 126 us, 4.2 TB/s) and with stochastic rounding the vector pipe.  A lane used to own all 32 rows of 8 columns (171 - 188 registers, two
// wavefronts per SIMD; now 110 - 128 and four), us per call: X 4096 x 5120 28.7 -> 21.4, with stochastic rounding 41.5 -> 28.1; X 8192 x 5120 43.6 -> 34.7,
// 60.6 -> 47.2; 8192 x 20480 149 -> 129, 198 -> 154; 256 x 512 11.0 -> 7.1, 14.2 -> 9.0.  A block's power of two as the conversions' scale
// operand instead of a multiplication per value, and its byte from two integer operations: 4096 x 5120 21.0 -> 19.2, 28.6 -> 26.9; 8192 x 20480 133 -> 126,
// 157 -> 151.
//
// Random draws: the row copy uses the NVFP4 draws (counter (j / 8, i, 0, 0)); the
// col copy draws its own, counter (i / 8, j, 1, 0), word (i % 8) / 2, low half for
// even i, so that eight consecutive rows of a column come from one Philox call.
#include "nvfp4_internal.h"
#include "nvfp4_device.h"

namespace nvfp4 {

namespace {

constexpr int kThreads = 256;
constexpr int kTileCols = 256, kTileRows = 128;
constexpr int kSlot = 33;   // column octets per staging row, padded

// Eight values, divided by the power of two `scale` -> one dword of eight codes (value t in nibble t).  The division is the conversion's own: one multiplication per value less.
template <bool kSR>
__device__ __forceinline__ uint32_t encode8(const float v[8], float scale, const uint32_t draws_hi16[8]) {
  if (!kSR) {
    uint32_t d = any_word(v[0]);
    d = cvt_rne_pair<0>(d, v[0], v[1], scale);
    d = cvt_rne_pair<1>(d, v[2], v[3], scale);
    d = cvt_rne_pair<2>(d, v[4], v[5], scale);
    d = cvt_rne_pair<3>(d, v[6], v[7], scale);
    return d;
  } else {
    uint32_t e = any_word(v[0]), o = any_word(v[1]);
    cvt_sr_single_into<0>(e, v[0], draws_hi16[0], scale);
    cvt_sr_single_into<1>(e, v[2], draws_hi16[2], scale);
    cvt_sr_single_into<2>(e, v[4], draws_hi16[4], scale);
    cvt_sr_single_into<3>(e, v[6], draws_hi16[6], scale);
    cvt_sr_single_into<0>(o, v[1], draws_hi16[1], scale);
    cvt_sr_single_into<1>(o, v[3], draws_hi16[3], scale);
    cvt_sr_single_into<2>(o, v[5], draws_hi16[5], scale);
    cvt_sr_single_into<3>(o, v[7], draws_hi16[7], scale);
    return interleave_nibbles(e, o);
  }
}

// the eight 16-bit draws of one Philox call, each moved to the top half of a word
__device__ __forceinline__ void draws8(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t k0, uint32_t k1, uint32_t out[8]) {
  uint32_t w[4];
  philox4x32_10(c0, c1, c2, 0u, k0, k1, w);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    out[2 * t] = w[t] << 16;
    out[2 * t + 1] = w[t] & 0xFFFF0000u;
  }
}

__device__ __forceinline__ float elem(const uint4& q, int c) {
  const uint32_t w = (c < 2) ? q.x : (c < 4) ? q.y : (c < 6) ? q.z : q.w;
  return (c & 1) ? bf16_hi(w) : bf16_lo(w);
}

// v of this lane, v of the lane 32 on (or back)
__device__ __forceinline__ float max_of_halves(float v) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

// kSplit: the two copies are made by two sets of workgroups (blockIdx.z).
template <bool kRow, bool kCol, bool kRht, bool kSR, bool kSplit>
__global__ __launch_bounds__(kThreads, 4) void quantize_mx_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                                  int64_t ld, uint32_t sign_mask, uint32_t key0, uint32_t key1,
                                                                  uint8_t* __restrict__ row_codes, uint8_t* __restrict__ row_scales,
                                                                  float* __restrict__ row_ts, uint8_t* __restrict__ col_codes,
                                                                  uint8_t* __restrict__ col_scales, float* __restrict__ col_ts) {
  __shared__ __attribute__((aligned(16))) uint8_t st_col_codes[kCol ? 8 * 4 * kSlot * 16 : 16];   // [column of the lane][wavefront][lane % 32] x 16 bytes, 8 of each half
  __shared__ uint8_t st_col_scales[kCol ? 8 * 4 * 32 : 16];                                      // [column of the lane][wavefront][lane % 32]
  __shared__ __attribute__((aligned(16))) uint8_t st_row_scales[kRow ? kTileRows * 8 : 16];      // [row][8 blocks]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
  const int64_t colblk = static_cast<int64_t>(blockIdx.x) * kTileCols;
  const int64_t col0 = colblk + l32 * 8;
  const int64_t rowblk = static_cast<int64_t>(blockIdx.y) * kTileRows;
  const int row_in = wave * 32 + half * 16;   // the lane's first row within the tile
  const int64_t row0 = rowblk + row_in;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
    // MXFP4 has no tensor-level scale: s_dec = 1; the amax slot is not computed.
    if (kRow) { row_ts[0] = 1.0f; row_ts[1] = 0.0f; }
    if (kCol) { col_ts[0] = 1.0f; col_ts[1] = 0.0f; }
  }
  const bool active = col0 < cols && row0 < rows;   // cols and rows are multiples of 32: both halves of a block or none

  uint4 raw[16];
  if (active) {
#pragma unroll
    for (int r = 0; r < 16; ++r) raw[r] = *reinterpret_cast<const uint4*>(x + (row0 + r) * ld + col0);
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) raw[r] = make_uint4(0u, 0u, 0u, 0u);
  }

  const bool do_row = kRow && (!kSplit || blockIdx.z == 0), do_col = kCol && (!kSplit || blockIdx.z == 1);
  if (do_row) {
#pragma unroll   // fully: a partly unrolled loop indexes raw[] at run time, which puts the whole patch in scratch memory
    for (int r = 0; r < 16; ++r) {
      float v[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = elem(raw[r], c);
      float m = 0.0f;
#pragma unroll
      for (int c = 0; c < 8; ++c) m = fmaxf(m, fabsf(v[c]));
      m = fmaxf(m, lane_xor1(m));   // a 32-column block is four neighbouring lanes
      m = fmaxf(m, lane_xor2(m));
      const uint32_t sc = ue8m0_scale(m);
      uint32_t dr[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (kSR) draws8(static_cast<uint32_t>(col0 >> 3), static_cast<uint32_t>(row0 + r), 0u, key0, key1, dr);
      const uint32_t codes = encode8<kSR>(v, conversion_scale(sc), dr);
      if (active) {
        *reinterpret_cast<uint32_t*>(row_codes + (row0 + r) * (cols / 2) + col0 / 2) = codes;
        if ((lane & 3) == 0) st_row_scales[(row_in + r) * 8 + (l32 >> 2)] = static_cast<uint8_t>(sc);
      }
      // keep the scheduler from interleaving all rows' temporaries on top of the registers of the patch
      if ((r & 3) == 3 || kSR) __builtin_amdgcn_sched_barrier(0);
    }
  }

  if (kRow && kCol) {
    // Opaque to the optimiser (no instruction emitted): otherwise it recognises the row pass's unpacked values
    // in the column pass and keeps all of them alive on top of the registers of the patch.
#pragma unroll
    for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(raw[r].x), "+v"(raw[r].y), "+v"(raw[r].z), "+v"(raw[r].w));
  }
  if (do_col) {
    if (kRht) {   // the sign diagonal, on two columns at a time
      const uint32_t signs = half ? sign_mask >> 16 : sign_mask;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t flip = (0u - (signs >> r & 1u)) & 0x80008000u;
        raw[r].x ^= flip, raw[r].y ^= flip, raw[r].z ^= flip, raw[r].w ^= flip;
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      // w[0 .. 15]: the lane's rows; with a rotation, after the exchange: w[i], w[i + 8] = rows i and i + 16 (lower half) or i + 8 and i + 24 (upper)
      float w[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) w[r] = elem(raw[r], c);
      if (kRht) {
#pragma unroll
        for (int h = 1; h < 16; h <<= 1) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            if ((i & h) == 0) {
              const float a = w[i], b = w[i + h];
              w[i] = a + b;
              w[i + h] = a - b;
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(w[i]), __float_as_uint(w[i + 8]), false, false);
          const float a = __uint_as_float(s[0]), b = __uint_as_float(s[1]);
          w[i] = 0.176776695296636893f * (a + b);
          w[i + 8] = 0.176776695296636893f * (a - b);
        }
      }
      float m = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, fabsf(w[r]));
      m = max_of_halves(m);
      const uint32_t sc = ue8m0_scale(m);
      uint2 out;
#pragma unroll
      for (int g = 0; g < 2; ++g) {   // eight consecutive rows each: groups half and half + 2 of the block's four, unrotated 2 half and 2 half + 1
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = w[8 * g + t];
        uint32_t dr[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int group = kRht ? half + 2 * g : 2 * half + g;
        if (kSR) draws8(static_cast<uint32_t>((rowblk >> 3) + wave * 4 + group), static_cast<uint32_t>(col0 + c), 1u, key0, key1, dr);
        (g ? out.y : out.x) = encode8<kSR>(v, conversion_scale(sc), dr);
      }
      *reinterpret_cast<uint2*>(st_col_codes + ((c * 4 + wave) * kSlot + l32) * 16 + half * 8) = out;
      if (half == 0) st_col_scales[(c * 4 + wave) * 32 + l32] = static_cast<uint8_t>(sc);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();

  const int tile_cols = static_cast<int>(cols - colblk < kTileCols ? cols - colblk : kTileCols);
  const int tile_groups = static_cast<int>((rows - rowblk < kTileRows ? rows - rowblk : kTileRows) / 32);   // 32-row groups in this tile
  if (do_row && tid < kTileRows) {
    // 128 rows x (tile_cols / 32) scale bytes; a full tile row is 8 contiguous bytes
    const int64_t row = rowblk + tid;
    if (row < rows) {
      const uint8_t* src = st_row_scales + tid * 8;
      uint8_t* dst = row_scales + row * (cols / 32) + colblk / 32;
      const int nb = tile_cols / 32;
      if (nb == 8 && ((cols / 32) & 7) == 0) {
        *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(src);
      } else {
        for (int b = 0; b < nb; ++b) dst[b] = src[b];
      }
    }
  }
  if (do_col) {
    const int64_t code_ld = rows / 2, scale_ld = rows / 32;
    const bool wide = (code_ld & 15) == 0;
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
      const int q = i * kThreads + tid;   // 1024 pieces of 16 bytes: column j, 32-row group g
      const int j = q >> 2, g = q & 3;
      if (j >= tile_cols || g >= tile_groups) continue;
      const int lj = j >> 3, c = j & 7;
      uint4 v = *reinterpret_cast<const uint4*>(st_col_codes + ((c * 4 + g) * kSlot + lj) * 16);
      if (kRht) v = make_uint4(v.x, v.z, v.y, v.w);   // staged as groups 0, 2 | 1, 3
      uint8_t* dst = col_codes + (colblk + j) * code_ld + (rowblk + 32 * g) / 2;
      if (wide) {
        *reinterpret_cast<uint4*>(dst) = v;
      } else {
        reinterpret_cast<uint32_t*>(dst)[0] = v.x;
        reinterpret_cast<uint32_t*>(dst)[1] = v.y;
        reinterpret_cast<uint32_t*>(dst)[2] = v.z;
        reinterpret_cast<uint32_t*>(dst)[3] = v.w;
      }
    }
    if (tid < tile_cols) {   // one column: up to 4 scale bytes
      const int lj = tid >> 3, c = tid & 7;
      uint8_t* dst = col_scales + (colblk + tid) * scale_ld + rowblk / 32;
      uint8_t sc[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) sc[g] = st_col_scales[(c * 4 + g) * 32 + lj];
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

template <bool kRow, bool kCol, bool kRht>
void dispatch(const QuantizeArgs& a, dim3 grid, hipStream_t s) {
  // Up to 640 workgroups (768 with stochastic rounding; 1024 are resident at once) the call takes as long as a patch or two do: each copy gets workgroups of its
  // own, though the patch is then read twice.  us, one set / two: X 4096 x 4096 (512) 17.7 / 16.4, X 4096 x 5120 (640) 22.4 / 20.7, without rotation 18.7 /
  // 17.1; X 4192 x 5120 (660) 24.3 / 26.3, 22.1 / 27.8; X 4096 x 6144 (768) 24.2 / 25.8, 20.5 / 23.7; with stochastic rounding 4096 x 5120 31.4 / 27.0, 4192 x
  // 5120 33.6 / 33.0, 4096 x 6144 32.9 / 32.0, 5120 x 6144 (960) 40.1 / 40.4.
  constexpr bool kBoth = kRow && kCol;
  const bool split = kBoth && static_cast<int64_t>(grid.x) * grid.y <= (a.sr ? 768 : 640);
  if (split) grid.z = 2;
  const auto kernel = a.sr ? (split ? &quantize_mx_kernel<kRow, kCol, kRht, true, kBoth> : &quantize_mx_kernel<kRow, kCol, kRht, true, false>)
                           : (split ? &quantize_mx_kernel<kRow, kCol, kRht, false, kBoth> : &quantize_mx_kernel<kRow, kCol, kRht, false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, static_cast<const uint16_t*>(a.x), a.rows, a.cols, a.ld, a.sign_mask, a.key0,
                     a.key1, a.row_codes, a.row_scales, a.row_ts, a.col_codes, a.col_scales, a.col_ts);
}

}  // namespace

hipError_t launch_quantize_mx(const QuantizeArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>((a.cols + kTileCols - 1) / kTileCols),
                  static_cast<unsigned>((a.rows + kTileRows - 1) / kTileRows));
  if (a.want_row && a.want_col) {
    if (a.rht) dispatch<true, true, true>(a, grid, s); else dispatch<true, true, false>(a, grid, s);
  } else if (a.want_row) {
    dispatch<true, false, false>(a, grid, s);
  } else {
    if (a.rht) dispatch<false, true, true>(a, grid, s); else dispatch<false, true, false>(a, grid, s);
  }
  return hipGetLastError();
}

}  // namespace nvfp4
