// Block-scaled GEMM straight from the packed codes for gfx950 (App. B.3 Eq. 5): no scratch, any K that is a multiple of
// 16.  The form for products that do not fill the chip with 256 x 256 tiles -- few tokens, small layers -- and for
// contraction lengths that are not a multiple of 64.
//
// A wavefront owns MB x NB blocks of 16 x 16 outputs and every WK-th window of 128 or 256 k; the WK wavefronts of a workgroup own
// the same outputs and add their sums through LDS at the end (WK = 1: they own different ones).  No barrier in the loop: a wavefront loads the codes and
// scales of its own rows into registers two windows ahead, passes them through its own piece of LDS, decodes them to FP16
// (value * block scale, exact) and feeds the 16x16x32 MFMA.
//   - Through LDS, because a load in the MFMA's lane order (16 consecutive lanes = 16 rows) touches 16 cache lines per 16
//     lanes; eight lanes to a row's 128 bytes (four to 64) touch 2 (4).  64 x 20480 x 5120: 35 us without this detour, 27 with.
//   - What bounds it is the issue of vector instructions: a 16 x 32 fragment takes 8 of them (4 cvt, 4 pk_mul) and serves MB or
//     NB MFMAs.  Measured, cycles per MFMA with V such instructions beside it: 8 + 4.5 V (16 alone), whichever wavefront of the SIMD they
//     are from, so that 4 x 4 blocks (V = 4) cannot do better than 26 and 8 x 5 (2.6) reach 20: the large shapes have one wavefront per SIMD
//     and 320 to 512 registers.
//   - One wavefront per SIMD has nobody to fill its waits, so the loop is pipelined: behind a row of MFMAs go the decode of the next row's
//     fragment, the LDS reads of the next step, the stores of the next window into LDS and the loads of the window after it, each
//     an instruction or two behind an MFMA (interleave).  64 x 80 tiles of 64 x 20480 x 8192: 30.7 us with the same parts in turn, 25.5 so;
//     128 x 80 tiles of 128 x 20480 x 8192 51.5 and 39.7.  Taken out one at a time (us of the 15.9 that 4096 k cost there): loads 2.6, LDS 0, both and
//     decode 6.7.
//   - Windows of 256 k, that is whole 128-byte lines of codes, need 40 % less time for the loads alone than 64-byte pieces (8.1 and 4.9 us at
//     64 x 20480 x 5120) and half the loads of scales; the small shapes, which share short K among many wavefronts, take 128.
// Decoding A once per workgroup and sharing it through LDS needs a barrier per step and was slower (33 against 22 us, 52 against 38).
// Measured (us; before = steps of 128 k in turn, at most 64 x 64 per wavefront): 64 x 20480 x 5120 23.5 -> 19.1, 128 x 20480 x 5120 39.8 -> 28.0, 512 x 5120 x
// 5120 39.3 -> 27.4, 1040 x 1296 x 2064 14.7 -> 13.1, 2064 x 1296 x 1040 15.8 -> 13.3, 8176 x 5104 x 5136 571 -> 395 (1.09 PFLOP/s).

#include <cmath>
#include <type_traits>
#include <utility>

#include "nvfp4_internal.h"
#include "nvfp4_device.h"
#include "gemm_epilogue.h"

namespace nvfp4 {
namespace {

struct __attribute__((packed, aligned(8))) Codes16 { uint32_t w[4]; };
typedef uint16_t u16_any __attribute__((aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));

// What a lane holds of a 16-row block and a window of 128 kSteps k as loaded: 16-byte chunk lane % (4 kSteps) (32 codes) of row
// lane / (4 kSteps), with two steps that of the row 8 below too, and the 2 kSteps scales lane % 4 of row lane / 4.
template <int kSteps>
struct Loaded {
  uint4 c[kSteps];
  uint32_t s;
};

__device__ __forceinline__ uint32_t word(const uint4& c, int t) { return t == 0 ? c.x : t == 1 ? c.y : t == 2 ? c.z : c.w; }

// 8 codes of k 8 t .. 8 t + 7 of a 32-code chunk, times the scale of their block
__device__ __forceinline__ half8v decode_part(const uint4& c, half2v scales, int t) {
  const _Float16 s = (t >> 1) ? scales.y : scales.x;
  return decode8_f16(word(c, t), half2v{s, s});
}
// Between lanes that exchange data through their wavefront's own piece of LDS: the hardware executes a wavefront's LDS
// instructions in order, so nothing has to be waited for, but the compiler must not move a read above the other lanes' writes
// (or a write above their reads) because it finds the addresses of one lane different.  No instruction.
__device__ __forceinline__ void wavefront_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int kBegin, int kEnd, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kBegin < kEnd) {
    f(std::integral_constant<int, kBegin>{});
    static_for<kBegin + 1, kEnd>(f);
  }
}

// The instructions since the last such call, in this order: the MFMAs with the others spread evenly behind them.
template <int kMfmas, int kValu, int kDsReads, int kDsWrites, int kLoads>
__device__ __forceinline__ void interleave() {
  static_for<0, kMfmas>([](auto n) {
    constexpr int g = decltype(n)::value;
    constexpr auto share = [](int total) { return (g + 1) * total / kMfmas - g * total / kMfmas; };
    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
    if constexpr (share(kDsReads) > 0) __builtin_amdgcn_sched_group_barrier(0x100, share(kDsReads), 0);
    if constexpr (share(kDsWrites) > 0) __builtin_amdgcn_sched_group_barrier(0x200, share(kDsWrites), 0);
    if constexpr (share(kLoads) > 0) __builtin_amdgcn_sched_group_barrier(0x20, share(kLoads), 0);
    if constexpr (share(kValu) > 0) __builtin_amdgcn_sched_group_barrier(0x2, share(kValu), 0);
  });
  __builtin_amdgcn_sched_barrier(0);
}

// MB x NB blocks of 16 x 16 outputs per wavefront, WK wavefronts per workgroup that split K.  WK = 1: a workgroup of 2 x 2
// wavefronts that own a tile each.  kSteps: a window is 128 or 256 k.
template <int MB, int NB, int WK, int Steps>
struct Shape {
  static constexpr int kOwn = WK == 1 ? 2 : 1, kWaves = WK * kOwn * kOwn;
  static constexpr int kTM = MB * 16 * kOwn, kTN = NB * 16 * kOwn, kThreads = kWaves * 64, kBlocks = MB + NB;
  static constexpr int kSteps = Steps, kWindowK = 128 * kSteps;
  static constexpr int kCodeBytes = 16 * kWindowK / 2, kScaleBytes = kWindowK;   // of a 16-row block and window
  static constexpr int kStage = kBlocks * (kCodeBytes + kScaleBytes);            // a window's codes and scales, per wavefront
  static constexpr int kSum = WK > 1 ? MB * NB * 1024 : 0;
  static constexpr int kWaveBytes = kStage > kSum ? kStage : kSum;
  static constexpr int kLdsBytes = kWaves * kWaveBytes;
};

// Tile number pid of a product of tiles_m x tiles_n of them.  bf16_out: the output type, a constant where a kernel serves one.
template <int MB, int NB, int WK, int Steps>
__device__ __forceinline__ void direct_tile(const Operand& A, const Operand& B, const int K, void* __restrict__ Dv, const int64_t ldd, const bool accumulate,
                                            const bool bf16_out, const int tiles_m, const int tiles_n, int pid) {
  using S = Shape<MB, NB, WK, Steps>;
  constexpr int kSteps = Steps, kWindowK = S::kWindowK, kCodeBytes = S::kCodeBytes, kScaleBytes = S::kScaleBytes;
  constexpr int kChunks = 4 * kSteps, kLoadRows = 64 / kChunks, kRowBytes = 16 * kChunks;   // of a row of a window; rows that a load instruction covers
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6), wk = WK == 1 ? 0 : wave;
  const int num_tiles = tiles_m * tiles_n;
  if ((num_tiles & 7) == 0) pid = (pid & 7) * (num_tiles >> 3) + (pid >> 3);
  int tm, tn;
  tile_coordinates(pid, tiles_m, tiles_n, tm, tn);
  const int l16 = lane & 15, q = lane >> 4;
  const int crow = lane / kChunks, chunk = lane % kChunks, srow = lane >> 2, spart = lane & 3;   // loading: row and chunk of the lane's codes, of its scales
  // (unsigned: the last tile may reach past 2^31)
  const uint32_t M = static_cast<uint32_t>(A.outer), N = static_cast<uint32_t>(B.outer);
  const uint32_t m0 = tm * S::kTM + (WK == 1 ? (wave >> 1) * (MB * 16) : 0), n0 = tn * S::kTN + (WK == 1 ? (wave & 1) * (NB * 16) : 0);
  uint8_t* const mine = lds + wave * S::kWaveBytes;

  // Wave-uniform bases plus one 32-bit lane offset; blocks 0 .. MB-1 are A's, the others B's.  Blocks past the
  // end of an operand are replaced by its last (they feed outputs that are never stored).
  const int code_ld = K / 2, scale_ld = K / 16;
  const uint8_t *cp[S::kBlocks], *sp[S::kBlocks];
#pragma unroll
  for (int i = 0; i < S::kBlocks; ++i) {
    const int64_t row = i < MB ? min(m0 + i * 16u, M - 16u) : min(n0 + (i - MB) * 16u, N - 16u);
    cp[i] = (i < MB ? A.codes : B.codes) + row * code_ld;
    sp[i] = (i < MB ? A.scales : B.scales) + row * scale_ld;
  }
  const uint32_t code_off = static_cast<uint32_t>(crow * code_ld + chunk * 16), scale_off = static_cast<uint32_t>(srow * scale_ld + spart * 2 * kSteps);

  // The wavefront's part of K: every WK-th window, and one of them the rest.  (A stretch of K to each, as even as 64 k allow, was slower, also where
  // the windows do not come out even: neighbouring lines then go to one wavefront one after the other.  512 x 5120 x 5120 29.1 / 28.4 us, 1040 x 1296 x
  // 2064 13.7 / 13.1; with windows of 128, half a line, 32 x 5120 x 5120 7.6 / 7.1.)
  const int full = K / kWindowK, windows = (full - wk + WK - 1) / WK, rest = full % WK == wk ? K - full * kWindowK : 0;

  float4v acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

  Loaded<kSteps> ld[S::kBlocks];
  auto load_block = [&](int i, int k, const uint32_t (&co)[kSteps], uint32_t so) {
#pragma unroll
    for (int h = 0; h < kSteps; ++h) {
      const Codes16 w = *reinterpret_cast<const Codes16*>(cp[i] + k / 2 + co[h]);
      ld[i].c[h] = make_uint4(w.w[0], w.w[1], w.w[2], w.w[3]);
    }
    const uint8_t* from = sp[i] + k / 16 + so;
    ld[i].s = kSteps == 2 ? *reinterpret_cast<const u32_any*>(from) : *reinterpret_cast<const u16_any*>(from);
  };
  // the lane's offsets, or 0 where there is nothing to load (one line instead of 40).  Opaque (no instruction): otherwise the compiler
  // keeps every block's sum of base and offset as a 64-bit address in vector registers, more than there are.
  auto offsets = [&](bool any, uint32_t (&co)[kSteps], uint32_t& so) {
#pragma unroll
    for (int h = 0; h < kSteps; ++h) {
      co[h] = any ? code_off + static_cast<uint32_t>(h * kLoadRows * code_ld) : 0u;
      asm volatile("" : "+v"(co[h]));
    }
    so = any ? scale_off : 0u;
    asm volatile("" : "+v"(so));
  };
  auto load = [&](int k) {
    uint32_t co[kSteps], so;
    offsets(true, co, so);
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) load_block(i, k, co, so);
  };
  // The rest of K as a window of 128 that ends where K does, whose scales are 0 for what is not the rest's.
  auto load_rest = [&]() {
    load(K - kWindowK);
    const int first = (kWindowK - rest) / 16 - spart * 2;   // block of the rest's first k, counted from the lane's
    const uint32_t mask = first <= 0 ? 0xFFFFu : first == 1 ? 0xFF00u : 0u;
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) ld[i].s &= mask;
  };
  // K shorter than a window of 128: a lane's chunk, and its two scales, are there whole, half or not at all; what is not is read from the row's first
  // bytes, and its scales are 0.  The offsets and the mask are opaque (no instruction): knowing that they go together the compiler jumps around each
  // block's scales and waits for them there, one block after the other (4096 x 304 x 112 5.5 us, 4.9 so).
  auto load_short = [&]() {
    const bool in0 = chunk * 32 < K, in1 = chunk * 32 + 16 < K;
    uint32_t lo = static_cast<uint32_t>(crow * code_ld) + (in0 ? chunk * 16 : 0), hi = lo + (in1 ? 8 : 0);
    uint32_t s0 = static_cast<uint32_t>(crow * scale_ld) + (in0 ? chunk * 2 : 0), s1 = s0 + (in1 ? 1 : 0), mask = (in0 ? 0xFFu : 0u) | (in1 ? 0xFF00u : 0u);
    asm volatile("" : "+v"(lo), "+v"(hi), "+v"(s0), "+v"(s1), "+v"(mask));
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) {
      const uint2 c_lo = *reinterpret_cast<const uint2*>(cp[i] + lo), c_hi = *reinterpret_cast<const uint2*>(cp[i] + hi);
      ld[i].c[0] = make_uint4(c_lo.x, c_lo.y, c_hi.x, c_hi.y);
      ld[i].s = (sp[i][s0] | static_cast<uint32_t>(sp[i][s1]) << 8) & mask;
    }
    asm volatile("");   // (or the loads are merged with load()'s, in pieces and with addresses in vector registers)
  };
  // The window in hand through LDS: stored as loaded, but chunk c of row r at position c ^ swizzle(r), read back in the MFMA's lane order: a
  // lane takes chunks kSteps q .. of its row, one in each step, of which each MFMA of the step takes 8 codes, and their scales.
  auto swizzle = [](int row) { return kSteps == 2 ? row & 7 : row >> 1 & 3; };   // eight consecutive rows of one chunk: all banks
  auto stage = [&](int i) {
#pragma unroll
    for (int h = 0; h < kSteps; ++h)   // (kLoadRows is a multiple of the swizzle's period)
      *reinterpret_cast<uint4*>(mine + i * kCodeBytes + (h * kLoadRows + crow) * kRowBytes + (chunk ^ swizzle(crow)) * 16) = ld[i].c[h];
    uint8_t* const to = mine + S::kBlocks * kCodeBytes + i * kScaleBytes + lane * 2 * kSteps;
    if (kSteps == 2) *reinterpret_cast<uint32_t*>(to) = ld[i].s;
    else *reinterpret_cast<uint16_t*>(to) = static_cast<uint16_t>(ld[i].s);
  };
  const uint8_t* const my_codes = mine + l16 * kRowBytes;
  const uint8_t* const my_scales = mine + S::kBlocks * kCodeBytes + l16 * (8 * kSteps);
  const uint32_t at0 = static_cast<uint32_t>((kSteps * q) ^ swizzle(l16)) << 4;   // of chunk kSteps q; kSteps q + 1 is at at0 ^ 16
  uint4 c[S::kBlocks];
  uint32_t raw[S::kBlocks];   // the scales of the window
  half2v sc[S::kBlocks];      // the 2 of the step
  half8v f[2][S::kBlocks];
  auto read_codes = [&](int i, int step) { c[i] = *reinterpret_cast<const uint4*>(my_codes + i * kCodeBytes + (at0 ^ (step * 16))); };
  auto read_scales = [&](int i) {
    const uint8_t* from = my_scales + i * kScaleBytes + q * 2 * kSteps;
    raw[i] = kSteps == 2 ? *reinterpret_cast<const uint32_t*>(from) : *reinterpret_cast<const uint16_t*>(from);
  };
  auto decode = [&](int i, int step, int t) {
    if (t == 0) sc[i] = step ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(raw[i]), 1.0f, true)
                             : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(raw[i]), 1.0f, false);
    f[t & 1][i] = decode_part(c[i], sc[i], t);
  };
  auto multiply_row = [&](int i, int t) {
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f[t & 1][MB + j], f[t & 1][i], acc[i][j], 0, 0, 0);
  };
  // The part of [0, total) that falls to place n of `places`
  constexpr auto part = [](int n, int total, int places) { return n * total / places; };
  // One window, whose first step's codes and scales are in c and raw and its first fragments decoded: f[0] of A's block 0 and of all of B's.
  // kSteps steps x 4 fragments of depth 32 x MB rows of MFMAs.  Behind a row's MFMAs: the next row's fragment of A, a share of the next
  // depth's of B; in the last depth of a step the reads of the next step's codes, each as soon as the registers are free.
  // kMore: a next window follows: in the last step's first three depths it goes to LDS, block by block, and each block's loads of the window
  // after that are issued.
  auto run_window = [&](auto more, int k_load, const uint32_t (&co)[kSteps], uint32_t so) {
    constexpr bool kMore = decltype(more)::value;
    static_for<0, 4 * kSteps * MB>([&](auto n) {
      constexpr int at = decltype(n)::value, step = at / (4 * MB), t = at / MB % 4, i = at % MB;
      constexpr bool last_step = step == kSteps - 1, next_step = !last_step || kMore;   // after depth 3: is there one
      constexpr int to_step = last_step ? 0 : step + 1;
      constexpr int kFirst = MB > 2 ? 2 : MB - 1;         // row of depth 3 from which B's next fragments are decoded: the reads are back
      // reads of the next step, in depth 3: all of B's blocks and A's first in row 0, then A's block by block
      if constexpr (t == 3 && next_step) {
        if constexpr (i == 0) {
          if constexpr (last_step) wavefront_exchange();
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            read_codes(MB + b, to_step);
            if (last_step) read_scales(MB + b);
          }
        }
        read_codes(i, to_step);
        if (last_step) read_scales(i);
        if constexpr (i == MB - 1) wavefront_exchange();   // the next window's stores come after these reads
      }
      constexpr int reads = t == 3 && next_step ? ((i == 0 ? NB : 0) + 1) * (last_step ? 2 : 1) : 0;
      if constexpr (i + 1 < MB) decode(i + 1, step, t);
      else if constexpr (t < 3) decode(0, step, t + 1);
      else if constexpr (next_step) decode(0, to_step, 0);
      constexpr bool a_here = i + 1 < MB || t < 3 || next_step;
      constexpr int b0 = t < 3 ? part(i, NB, MB) : i < kFirst || !next_step ? 0 : part(i - kFirst, NB, MB - kFirst);
      constexpr int b1 = t < 3 ? part(i + 1, NB, MB) : i < kFirst || !next_step ? 0 : part(i + 1 - kFirst, NB, MB - kFirst);
#pragma unroll
      for (int b = b0; b < b1; ++b) {
        if (t < 3) decode(MB + b, step, t + 1);
        else decode(MB + b, to_step, 0);
      }
      constexpr bool staging = kMore && last_step && t < 3;
      constexpr int place = t * MB + i, s0 = staging ? part(place, S::kBlocks, 3 * MB) : 0, s1 = staging ? part(place + 1, S::kBlocks, 3 * MB) : 0;
#pragma unroll
      for (int b = s0; b < s1; ++b) {
        stage(b);
        load_block(b, k_load, co, so);
      }
      multiply_row(i, t);
      interleave<NB, (a_here ? 8 : 0) + 8 * (b1 - b0), reads, (1 + kSteps) * (s1 - s0), (1 + kSteps) * (s1 - s0)>();
    });
  };
  // 8 codes per lane of every block, k .. k + 31 of the window, in f[t]; blocks of 16 below lo count for nothing
  auto rest_piece = [&](int k, int lo, int t) {
    const int at = k + q * 8, block = at >> 4;
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) {
      const uint32_t w = *reinterpret_cast<const uint32_t*>(my_codes + i * kCodeBytes + (((at >> 5) ^ swizzle(l16)) << 4) + (at >> 3 & 3) * 4);
      const uint32_t s = my_scales[i * kScaleBytes + block];
      f[t][i] = decode8_f16(w, e4m3_decode_f16x2(block * 16 >= lo ? s : 0u));
    }
  };
  // The rest: the first of the wavefront's windows, or the last, in pieces of 32 k of which nothing overlaps: with windows of 256, and up to 64 k in the
  // larger tiles, where a window would leave more than half of it empty.  us, window / pieces: 64 x 64 tiles of 320 x 2560 x 368 5.1 / 5.4, 64 x 48 of 448 x
  // 1456 x 368 4.6 / 4.9, 16 x 32 of 48 x 768 x 4272 5.7 / 5.8; own 64 x 64 of 304 x 20224 x 144 12.2 / 11.4, 64 x 64 of 1344 x 1536 x 192 6.3 / 6.0.
  constexpr bool kAlwaysFirst = kSteps == 1 && MB * NB <= 4;
  const bool rest_first = kAlwaysFirst || (kSteps == 1 && (rest > 64 || full == 0)), pieces = !rest_first && rest;
  const int total = windows + (rest ? 1 : 0);
  if (total) {
    const int first = rest_first && rest ? wk - WK : wk;   // number of the window that would be the first if all were whole
    auto k_of = [&](int n) { return rest_first || n < windows ? (first + n * WK) * kWindowK : K - kWindowK; };
    if (!rest_first || !rest) load(k_of(0));
    else if constexpr (kSteps == 1) {
      if (full) load_rest();
      else load_short();
    }
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) stage(i);
    wavefront_exchange();
    if (rest_first || windows) {
      if (total > 1) load(k_of(1));
#pragma unroll
      for (int i = 0; i < S::kBlocks; ++i) {
        read_codes(i, 0);
        read_scales(i);
      }
      decode(0, 0, 0);
#pragma unroll
      for (int b = 0; b < NB; ++b) decode(MB + b, 0, 0);
#pragma unroll 1
      for (int next = 1; next < total; ++next) {
        uint32_t co[kSteps], so;
        offsets(next + 1 < total, co, so);
        run_window(std::true_type{}, k_of(min(next + 1, total - 1)), co, so);
      }
      if (kAlwaysFirst || !pieces) run_window(std::false_type{}, 0, {}, 0u);
    }
    if (!kAlwaysFirst && pieces) {
      const int lo = kWindowK - rest;
      int hi = kWindowK;
      if (static_cast<unsigned>(hi - lo - 1) % 64 < 32) {
        hi -= 32;
        rest_piece(hi, lo, 0);
#pragma unroll
        for (int i = 0; i < MB; ++i) multiply_row(i, 0);
      }
#pragma unroll 1
      for (hi -= 64; hi > lo - 64; hi -= 64) {
        rest_piece(hi, lo, 0);
        rest_piece(hi + 32, lo, 1);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < MB; ++i) multiply_row(i, t);
      }
    }
  }

  const TensorScales ts{A.ts, B.ts, A.ts_per_row != 0, B.ts_per_row != 0};
  const bool vec = ts.a_per_row || ts.b_per_row;
  const float out_scale = vec ? 0.0f : A.ts[0] * B.ts[0];
  auto store = [&](float4v v, int i, int j) {
    const uint32_t m = m0 + i * 16 + l16, n = n0 + j * 16 + q * 4;
    if (m < M && n < N) {
      v *= scale4(ts, out_scale, vec, true, m, n);
      if (bf16_out) {
        uint2 o;
        o.x = f32x2_to_bf16(v[0], v[1]);
        o.y = f32x2_to_bf16(v[2], v[3]);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(Dv) + m * ldd + n) = o;
      } else {
        float* d = static_cast<float*>(Dv) + m * ldd + n;
        if (accumulate) v += *reinterpret_cast<const float4v*>(d);
        *reinterpret_cast<float4v*>(d) = v;
      }
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) store(acc[i][j], i, j);
  } else {
    constexpr int kFrags = MB * NB;
    __syncthreads();   // everybody is done with the staged operands
#pragma unroll
    for (int f = 0; f < kFrags; ++f) reinterpret_cast<float4v*>(mine)[f * 64 + lane] = acc[f / NB][f % NB];
    __syncthreads();
    for (int f = wk; f < kFrags; f += WK) {
      const uint8_t* p = lds + (f * 64 + lane) * 16;
      float4v v = *reinterpret_cast<const float4v*>(p);
#pragma unroll
      for (int w = 1; w < WK; ++w) v += *reinterpret_cast<const float4v*>(p + w * S::kWaveBytes);
      store(v, f / NB, f % NB);
    }
  }
}

template <int MB, int NB, int WK, int Steps, bool kBf16Out>
__global__ __launch_bounds__((WK == 1 ? 4 : WK) * 64, MB * NB > 16 ? 1 : 2) void gemm_direct_kernel(
    Operand A, Operand B, int K, void* __restrict__ Dv, int64_t ldd, bool accumulate, int tiles_m, int tiles_n) {
  direct_tile<MB, NB, WK, Steps>(A, B, K, Dv, ldd, accumulate, kBf16Out, tiles_m, tiles_n, static_cast<int>(blockIdx.x));
}

// Two products that do not depend on each other in one launch (a layer's Dgrad and Wgrad): the first `tiles` workgroups take the first one's tiles.  Apart, a small layer's
// products leave the chip half empty one after the other: 1040 x 2064 x 1296 has 731 tiles for 512 places, 2064 x 1296 x 1040 187.  Each is worked
// exactly as by a launch of its own.  The shapes are those of which two workgroups of four wavefronts fit a CU.  Backward calls (quantizer included), us, apart / in one launch:
// tokens x d_in x d_out 1040 x 2064 x 1296 42.0 / 37.1, 416 x 1280 x 512 16.8 / 13.7, 240 x 2304 x 16384 94.5 / 82.3, 6912 x 448 x 13664 338 / 328; geometric mean
// over 100 sizes 1.09; where two launches are faster: direct_pair_pays.  The product with the shorter wavefronts first: 1.07.
struct DirectProduct {
  Operand a, b;
  void* d;
  int64_t ldd;
  int K, tiles_m, tiles_n, shape;   // shape: 0 64 x 64 and 1 64 x 48 with K split, 2 64 x 64 to each wavefront
  bool accumulate, bf16_out;
};
__global__ __launch_bounds__(256, 2) void gemm_direct_pair_kernel(DirectProduct first, DirectProduct second) {
  const int tiles = first.tiles_m * first.tiles_n, id = static_cast<int>(blockIdx.x);
  const DirectProduct& p = id < tiles ? first : second;
  const int pid = id < tiles ? id : id - tiles;
  if (p.shape == 0) direct_tile<4, 4, 4, 1>(p.a, p.b, p.K, p.d, p.ldd, p.accumulate, p.bf16_out, p.tiles_m, p.tiles_n, pid);
  else if (p.shape == 1) direct_tile<4, 3, 4, 1>(p.a, p.b, p.K, p.d, p.ldd, p.accumulate, p.bf16_out, p.tiles_m, p.tiles_n, pid);
  else direct_tile<4, 4, 1, 1>(p.a, p.b, p.K, p.d, p.ldd, p.accumulate, p.bf16_out, p.tiles_m, p.tiles_n, pid);
}

}  // namespace

// The tile shapes the kernel comes in: MB x NB blocks per wavefront, WK wavefronts that split K, steps of 128 k to a window.  `kind` (for the
// tests): 0 16 x 32 tiles, 1 32 rows, 2 64 x 48 and 80 columns, 3 64 x 64 and 128 rows, 4 a tile to each wavefront.  Which of them: the smallest `us`, fitted,
// three constants to a shape, to products of 16 .. 8192 rows, 256 .. 20480 columns, K 16 .. 20480 (profiles/gemm_routes_us.csv; 5th and 95th
// percentile 0.83 and 1.16 of the measured time).  Large tiles decode less per product, small ones fill the chip; without a
// split of K there is no sum through LDS.  us, 64 x 48 / 64 x 64 / 64 x 80 / 128 x 80 / own 64 x 64 / own 128 x 80 / the rest at best: 64 x 20480 x 5120 22.1 /
// 26.1 / 19.0 / 27.6 / 42 / 84 / 20.3, 512 x 5120 x 5120 40 / 36 / 35 / 28 / 44 / 84 / 36, 4096 x 5120 x 2064 130 / 122 / 168 / 130 / 119 / 97 / 120,
// 1024 x 1024 x 1024 7.2 / 6.1 / 6.9 / 10 / 12 / - / 7.5, 32 x 5120 x 5120 12 / 13 / 16 / 24 / 41 / - / 7.1 (32 x 32).  What a shape earns, over the products
// of that table: without it they take so many % longer, the worst that many times as long (64 x 48 with windows of 256, 0.01 % and 1.12, went).
struct DirectShape {
  int mb, nb, wk, steps, kind;
  SmallTileCost us;
};
constexpr DirectShape kDirectShapes[] = {
    {4, 4, 4, 1, 3, {2, 1.12, 0.99, 1.06}},    // 1.16 %, 1.52
    {2, 2, 8, 1, 1, {2, 1.03, 0.27, 0.806}},   // 0.70 %, 1.62
    {4, 3, 4, 1, 2, {2, 1.13, 0.64, 0.934}},   // 0.81 %, 1.43
    {1, 2, 4, 1, 0, {5, 1.38, 0.08, 0.285}},   // 0.50 %, 1.45
    {1, 2, 4, 2, 0, {5, 1.53, 0.03, 0.26}},    // 0.18 %, 1.17
    {1, 2, 8, 1, 0, {3, 1.15, 0.11, 0.545}},   // 0.80 %, 1.32
    {2, 4, 8, 1, 1, {1, 1.0, 0.72, 1.46}},     // 0.34 %, 1.29
    {4, 5, 4, 2, 2, {1, 1.0, 1.89, 1.39}},     // 0.25 %, 1.43
    {5, 5, 4, 2, 2, {1, 1.0, 2.26, 1.6}},      // 0.20 %, 1.39
    {8, 5, 4, 2, 3, {1, 1.0, 3.51, 2.29}},     // 0.25 %, 1.34
    {4, 4, 1, 1, 4, {2, 1.08, 2.0, 1.03}},     // 0.98 %, 1.42
    {8, 5, 1, 2, 4, {1, 1.0, 8.07, 2.0}},      // 0.18 %, 1.57
    {6, 4, 1, 2, 4, {1, 1.0, 5.02, 1.38}},     // 0.17 %, 1.32
};
constexpr int kNumDirectShapes = sizeof(kDirectShapes) / sizeof(kDirectShapes[0]);
using AllShapes = std::make_integer_sequence<int, kNumDirectShapes>;

// (Shapes as template arguments: every division is by a constant.)
template <int I>
static int64_t direct_tiles(int64_t M, int64_t N) {
  constexpr DirectShape d = kDirectShapes[I];
  constexpr int tm = d.mb * (d.wk == 1 ? 32 : 16), tn = d.nb * (d.wk == 1 ? 32 : 16);
  return ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
}

// What the kernel's 32-bit rows, byte offsets within a 16-row block and launch size allow, and at least one window where it has 256 k (a shorter
// contraction leaves most of such a wavefront's loads empty); others take other kernels.
template <int I>
static bool fits(int64_t M, int64_t N, int64_t K) {
  constexpr DirectShape d = kDirectShapes[I];
  return M <= 0x7fffffff && N <= 0x7fffffff && K <= (int64_t{1} << 27) && (d.steps == 1 || K >= 128 * d.steps) &&
         direct_tiles<I>(M, N) * (d.wk == 1 ? 256 : d.wk * 64) <= 0xffffffff;
}

template <int... I>
static int64_t tiles_of(const GemmArgs& g, int shape, std::integer_sequence<int, I...>) {
  return ((shape == I ? direct_tiles<I>(g.a.outer, g.b.outer) : 0) + ...);
}
static int64_t tiles_of(const GemmArgs& g, int shape) { return tiles_of(g, shape, AllShapes{}); }

// Steps (128 k) of the wavefront that has most of them.  A rest that is worked in pieces counts half a step more than its k.
template <int I>
static double wavefront_steps(int64_t K) {
  constexpr DirectShape d = kDirectShapes[I];
  constexpr int window = 128 * d.steps;
  const int64_t full = K / window, rest = K - full * window, each = full / d.wk;
  const double whole = static_cast<double>((each + (full > each * d.wk)) * d.steps);
  const bool a_window = d.steps == 1 && (d.mb * d.nb <= 4 || rest > 64 || full == 0);
  const double with_rest = static_cast<double>(each * d.steps) + (rest ? (a_window ? 1.0 : 0.5 + static_cast<double>(rest) / 128.0) : 0.0);
  return whole > with_rest ? whole : with_rest;
}

// A tile to each wavefront and one workgroup to a CU: large results wait more for their stores, and accumulated ones for their loads, than two
// workgroups do: us, 64 x 64 / 128 x 80: 4096 x 8192 x 1040 93 / 114, accumulated 111 / 165; 6560 x 8320 x 1056 accumulated 189 / 223.
template <int I>
static double shape_loop_us(const GemmArgs& g, double elements) {
  if (!fits<I>(g.a.outer, g.b.outer, g.K)) return HUGE_VAL;
  constexpr DirectShape d = kDirectShapes[I];
  const double us = loop_us(d.us, direct_tiles<I>(g.a.outer, g.b.outer), wavefront_steps<I>(g.K));
  return d.wk == 1 && d.us.resident == 1 && elements > 3e7 ? 1.1 * us : us;
}

template <int... I>
static DirectPick pick_shape(const GemmArgs& g, bool split_only, std::integer_sequence<int, I...>) {
  const double elements = static_cast<double>(g.a.outer) * static_cast<double>(g.b.outer);
  DirectPick best{0, 0, HUGE_VAL};
  auto consider = [&](int shape, double us) {
    if (us < best.loop) best = DirectPick{shape, kDirectShapes[shape].kind, us};
  };
  (((split_only && kDirectShapes[I].wk == 1) ? void() : consider(I, shape_loop_us<I>(g, elements))), ...);
  return best;
}

DirectPick pick_direct_shape(const GemmArgs& g, bool split_only) { return pick_shape(g, split_only, AllShapes{}); }

bool direct_shape(int shape, int* out) {
  if (shape < 0 || shape >= kNumDirectShapes) return false;
  const DirectShape& d = kDirectShapes[shape];
  out[0] = d.mb, out[1] = d.nb, out[2] = d.wk, out[3] = d.steps;
  return true;
}

template <int I, bool kBf16Out>
static hipError_t launch_shape(const GemmArgs& g, hipStream_t s) {
  constexpr DirectShape d = kDirectShapes[I];
  using S = Shape<d.mb, d.nb, d.wk, d.steps>;
  constexpr auto kernel = &gemm_direct_kernel<d.mb, d.nb, d.wk, d.steps, kBf16Out>;
  static PerDeviceOnce once;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), S::kLdsBytes, once);
  if (e != hipSuccess) return e;
  const int tiles_m = static_cast<int>((g.a.outer + S::kTM - 1) / S::kTM), tiles_n = static_cast<int>((g.b.outer + S::kTN - 1) / S::kTN);
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(tiles_m * tiles_n)), dim3(S::kThreads), S::kLdsBytes, s, g.a, g.b, static_cast<int>(g.K), g.d,
                     g.ldd, g.accumulate, tiles_m, tiles_n);
  return hipGetLastError();
}

template <bool kBf16Out, int... I>
static hipError_t launch_direct(const GemmArgs& g, int shape, hipStream_t s, std::integer_sequence<int, I...>) {
  hipError_t e = hipErrorInvalidValue;
  ((shape == I ? void(e = launch_shape<I, kBf16Out>(g, s)) : void()), ...);
  return e;
}

template <int... I>
static bool fits_shape(const GemmArgs& g, int shape, std::integer_sequence<int, I...>) {
  return ((shape == I && fits<I>(g.a.outer, g.b.outer, g.K)) || ...);
}

bool direct_shape_fits(const GemmArgs& g, int shape) { return fits_shape(g, shape, AllShapes{}); }

// The pair kernel's number of a shape, or -1.
static int pair_shape(int shape) {
  const DirectShape& d = kDirectShapes[shape];
  if (d.mb != 4 || d.steps != 1) return -1;
  if (d.wk == 4) return d.nb == 4 ? 0 : d.nb == 3 ? 1 : -1;
  return d.wk == 1 && d.nb == 4 ? 2 : -1;
}

// Where one launch takes longer than two: one product has a tile for nearly every CU, the other between one and two.  Apart they come out even over the CUs; in one launch the
// places fall free unevenly, and a CU that gets two of the last tiles works at half the speed on each.  What that costs grows with the length of the tiles of the
// smaller product; the launch that is saved is 2.5 us.  Over 873 sizes 242 are such, and take 0.6 % longer in one launch (4416 x 384 x 9456 195 / 176 us in two, 3408 x 960 x 6768
// 201 / 192, but 8064 x 1024 x 1024 62 / 65); the others take 8 % less in one, the worst of them 1.7 % more.
bool direct_pair_pays(const GemmArgs& g, const DirectPick& p, const GemmArgs& h, const DirectPick& q) {
  const int64_t tg = tiles_of(g, p.shape), th = tiles_of(h, q.shape);
  const bool uneven = tg <= th ? tg > 192 && tg <= 256 && th > 256 && th <= 512 : th > 192 && th <= 256 && tg > 256 && tg <= 512;
  return !(uneven && (tg <= th ? p : q).loop > 10.0);
}

bool direct_pair_fits(const GemmArgs& g, int shape, const GemmArgs& h, int shape2) {
  if (pair_shape(shape) < 0 || pair_shape(shape2) < 0 || !direct_shape_fits(g, shape) || !direct_shape_fits(h, shape2)) return false;
  return tiles_of(g, shape) + tiles_of(h, shape2) <= 0xffffffff / 256;   // threads of a launch
}

// The product whose wavefronts run longer goes first, so that the other's fill the places that it leaves.
hipError_t launch_gemm_direct_pair(const GemmArgs& g, int shape, const GemmArgs& h, int shape2, hipStream_t s) {
  if (!direct_pair_fits(g, shape, h, shape2)) return hipErrorInvalidValue;
  auto product = [](const GemmArgs& x, int sh) {
    const DirectShape& d = kDirectShapes[sh];
    const int tm = d.mb * (d.wk == 1 ? 32 : 16), tn = d.nb * (d.wk == 1 ? 32 : 16);
    return DirectProduct{x.a, x.b, x.d, x.ldd, static_cast<int>(x.K), static_cast<int>((x.a.outer + tm - 1) / tm), static_cast<int>((x.b.outer + tn - 1) / tn),
                         pair_shape(sh), x.accumulate, x.out_bf16};
  };
  auto length = [](const GemmArgs& x, int sh) { return x.K / kDirectShapes[sh].wk * kDirectShapes[sh].nb; };
  DirectProduct first = product(g, shape), second = product(h, shape2);
  if (length(h, shape2) > length(g, shape)) std::swap(first, second);
  constexpr int lds = Shape<4, 4, 4, 1>::kLdsBytes;   // the most of the three
  static_assert(lds >= Shape<4, 3, 4, 1>::kLdsBytes && lds >= Shape<4, 4, 1, 1>::kLdsBytes, "");
  static PerDeviceOnce once;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_direct_pair_kernel), lds, once);
  if (e != hipSuccess) return e;
  const unsigned tiles = static_cast<unsigned>(first.tiles_m * first.tiles_n) + static_cast<unsigned>(second.tiles_m * second.tiles_n);
  hipLaunchKernelGGL(gemm_direct_pair_kernel, dim3(tiles), dim3(256), lds, s, first, second);
  return hipGetLastError();
}

hipError_t launch_gemm_direct(const GemmArgs& g, int shape, hipStream_t s) {
  if (!direct_shape_fits(g, shape)) return hipErrorInvalidValue;
  return g.out_bf16 ? launch_direct<true>(g, shape, s, AllShapes{}) : launch_direct<false>(g, shape, s, AllShapes{});
}

}  // namespace nvfp4
