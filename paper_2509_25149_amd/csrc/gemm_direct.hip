// Block-scaled GEMM straight from the packed codes for gfx950 (App. B.3 Eq. 5): no scratch, any K that is a multiple of
// 16.  The form for products that do not fill the chip with 256 x 256 tiles -- few tokens, small layers -- and for
// contraction lengths that are not a multiple of 64.
//
// A wavefront owns MB x NB blocks of 16 x 16 outputs and every WK-th step of 128 k; the WK wavefronts of a workgroup own
// the same outputs and add their sums through LDS at the end (WK = 1: they own different ones).  No barrier in the loop: a wavefront loads the codes and
// scales of its own rows into registers one step ahead, passes them through its own piece of LDS, decodes them to FP16
// (value * block scale, exact) and feeds the 16x16x32 MFMA.
//   - Through LDS, because a load in the MFMA's lane order (16 consecutive lanes = 16 rows) touches 16 cache lines per 16
//     lanes; four lanes to a row's 64 bytes touch 4.  64 x 20480 x 5120: 35 us without this detour, 27 with.
//   - Steps of 128 k rather than 256: half the LDS and the staging registers per wavefront, so that two workgroups of four
//     wavefronts fit a CU and the 427 of this shape are resident at once (27 -> 22 us), and less to lose where K is not a
//     multiple of the step.
//   - What bounds it is the issue of vector instructions: a 16 x 32 fragment takes 8 of them (4 cvt, 4 pk_mul) and serves MB or
//     NB (3 or 4) MFMAs, so the decode of the next fragments is spread over the MFMAs of these.  Decoding A once per
//     workgroup and sharing it through LDS needs a barrier per step and was slower (33 against 22 us, 52 against 38).
// Measured (us; before = whatever the call took then): 64 x 20480 x 5120 133 -> 23, 16 x 20480 x 5120 131 -> 14.6 (4.0 TB/s of
// codes), 512 x 5120 x 5120 101 -> 38, 256 x 256 x 512 18 -> 3.4, 1040 x 1296 x 2064 44 -> 14.4.

#include <cmath>

#include "nvfp4_internal.h"
#include "nvfp4_device.h"
#include "gemm_epilogue.h"

namespace nvfp4 {
namespace {

constexpr int kStepK = 128;               // k per step: 64 bytes of codes and 8 of scales per row, 1 KiB of codes per 16-row block
constexpr int kCodeBytes = 1024, kScaleBytes = 128;   // of a 16-row block and step

struct __attribute__((packed, aligned(8))) Codes16 { uint32_t w[4]; };
typedef uint16_t u16_any __attribute__((aligned(1)));

// What a lane holds of a 16-row block and step as loaded: row lane / 4, 16-byte chunk lane % 4 (32 codes), its 2 scales.
struct Loaded {
  uint4 c;
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
__device__ __forceinline__ half2v scales2(uint32_t s) { return __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(s), 1.0f, false); }

// MB x NB blocks of 16 x 16 outputs per wavefront, WK wavefronts per workgroup that split K.  WK = 1: a workgroup of 2 x 2
// wavefronts that own a tile each.
template <int MB, int NB, int WK>
struct Shape {
  static constexpr int kOwn = WK == 1 ? 2 : 1, kWaves = WK * kOwn * kOwn;
  static constexpr int kTM = MB * 16 * kOwn, kTN = NB * 16 * kOwn, kThreads = kWaves * 64, kBlocks = MB + NB;
  static constexpr int kStage = kBlocks * (kCodeBytes + kScaleBytes);       // one step's codes and scales, per wavefront
  static constexpr int kSum = WK > 1 ? MB * NB * 1024 : 0;
  static constexpr int kWaveBytes = kStage > kSum ? kStage : kSum;
  static constexpr int kLdsBytes = kWaves * kWaveBytes;
};

template <int MB, int NB, int WK, bool kBf16Out>
__global__ __launch_bounds__((WK == 1 ? 4 : WK) * 64, 2) void gemm_direct_kernel(Operand A, Operand B, int K, void* __restrict__ Dv, int64_t ldd,
                                                                  bool accumulate, int tiles_m, int tiles_n) {
  using S = Shape<MB, NB, WK>;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6), wk = WK == 1 ? 0 : wave;
  const int num_tiles = tiles_m * tiles_n;
  int pid = blockIdx.x;
  if ((num_tiles & 7) == 0) pid = (pid & 7) * (num_tiles >> 3) + (pid >> 3);
  int tm, tn;
  tile_coordinates(pid, tiles_m, tiles_n, tm, tn);
  const int l16 = lane & 15, q = lane >> 4;
  const int row4 = lane >> 2, c4 = lane & 3;      // loading: row and chunk of the lane
  const int M = static_cast<int>(A.outer), N = static_cast<int>(B.outer);
  const int m0 = tm * S::kTM + (WK == 1 ? (wave >> 1) * (MB * 16) : 0), n0 = tn * S::kTN + (WK == 1 ? (wave & 1) * (NB * 16) : 0);
  uint8_t* const mine = lds + wave * S::kWaveBytes;

  // Wave-uniform bases plus one 32-bit lane offset; blocks 0 .. MB-1 are A's, the others B's.  Blocks past the
  // end of an operand are replaced by its last (they feed outputs that are never stored).
  const int code_ld = K / 2, scale_ld = K / 16;
  const uint8_t *cp[S::kBlocks], *sp[S::kBlocks];
#pragma unroll
  for (int i = 0; i < S::kBlocks; ++i) {
    const int64_t row = i < MB ? min(m0 + i * 16, M - 16) : min(n0 + (i - MB) * 16, N - 16);
    cp[i] = (i < MB ? A.codes : B.codes) + row * code_ld;
    sp[i] = (i < MB ? A.scales : B.scales) + row * scale_ld;
  }
  const uint32_t code_off = static_cast<uint32_t>(row4 * code_ld + c4 * 16), scale_off = static_cast<uint32_t>(row4 * scale_ld + c4 * 2);

  float4v acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

  Loaded ld[S::kBlocks];
  auto load = [&](int i, int step) {
    const Codes16 c = *reinterpret_cast<const Codes16*>(cp[i] + step * 64 + code_off);
    ld[i].c = make_uint4(c.w[0], c.w[1], c.w[2], c.w[3]);
    ld[i].s = *reinterpret_cast<const u16_any*>(sp[i] + step * 8 + scale_off);
  };
  // The last, partial step (rest = 16 .. 112 k): a lane's chunk is whole, half there or absent; what is absent is read
  // from where the row still has bytes and gets scale 0.
  const int full = K / kStepK, rest = K - full * kStepK;
  auto load_tail = [&](int i) {
    const bool in0 = c4 * 32 < rest, in1 = c4 * 32 + 16 < rest;
    const uint32_t co = in0 ? code_off : code_off - c4 * 16, so = in0 ? scale_off : scale_off - c4 * 2;
    const uint2 lo = *reinterpret_cast<const uint2*>(cp[i] + full * 64 + co);
    const uint2 hi = *reinterpret_cast<const uint2*>(cp[i] + full * 64 + co + (in1 ? 8 : 0));
    const uint32_t s0 = sp[i][full * 8 + so], s1 = sp[i][full * 8 + so + (in1 ? 1 : 0)];
    ld[i].c = make_uint4(lo.x, lo.y, hi.x, hi.y);
    ld[i].s = (in0 ? s0 : 0u) | (in1 ? s1 << 8 : 0u);
  };
  // The step in hand through LDS: stored as loaded, read back in the MFMA's lane order.
  uint4 c[S::kBlocks];
  half2v sc[S::kBlocks];
  auto stage = [&](int i) {
    *reinterpret_cast<uint4*>(mine + i * kCodeBytes + (row4 * 4 + (c4 ^ (row4 >> 2))) * 16) = ld[i].c;
    *reinterpret_cast<uint16_t*>(mine + S::kBlocks * kCodeBytes + i * kScaleBytes + lane * 2) = static_cast<uint16_t>(ld[i].s);
  };
  auto read_back = [&](int i) {
    c[i] = *reinterpret_cast<const uint4*>(mine + i * kCodeBytes + (l16 * 4 + (q ^ (l16 >> 2))) * 16);
    sc[i] = scales2(*reinterpret_cast<const uint16_t*>(mine + S::kBlocks * kCodeBytes + i * kScaleBytes + l16 * 8 + q * 2));
  };
  // then: what else to issue on the way (the next step's loads).  With 8 blocks it goes between all the stores and all the reads (3328 x
  // 15856 x 4368 634 us, 660 block by block); with fewer a block is read back two blocks behind the stores, so that the first do not wait for the
  // last loads (64 x 20480 x 5120 23.7 us, 24.3 the other way).
  auto turn = [&](auto then) {
    if constexpr (S::kBlocks == 8) {
#pragma unroll
      for (int i = 0; i < S::kBlocks; ++i) stage(i);
      wavefront_exchange();
      then();
#pragma unroll
      for (int i = 0; i < S::kBlocks; ++i) read_back(i);
      wavefront_exchange();   // the next step's stores come after these reads
    } else {
      constexpr int kLag = 2;
#pragma unroll
      for (int i = 0; i < S::kBlocks + kLag; ++i) {
        if (i < S::kBlocks) {
          stage(i);
          wavefront_exchange();
        }
        if (i >= kLag) read_back(i - kLag);
      }
      wavefront_exchange();
      then();
    }
  };
  auto multiply = [&]() {
    half8v f[2][S::kBlocks];
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) f[0][i] = decode_part(c[i], sc[i], 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < 3) {
#pragma unroll
        for (int i = 0; i < S::kBlocks; ++i) f[(t + 1) & 1][i] = decode_part(c[i], sc[i], t + 1);
      }
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f[t & 1][MB + j], f[t & 1][i], acc[i][j], 0, 0, 0);
      if (t < 3) {   // the next fragments' decode spread over these MFMAs
        constexpr int kValu = (S::kBlocks * 8 + MB * NB - 1) / (MB * NB);
#pragma unroll
        for (int g = 0; g < MB * NB; ++g) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);
        }
      }
    }
  };
  const bool tail = rest && full % WK == wk;
  if (tail) {
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) load_tail(i);
    turn([] {});
  }
  if (wk < full) {
#pragma unroll
    for (int i = 0; i < S::kBlocks; ++i) load(i, wk);
  }
  if (tail) multiply();
#pragma unroll 1
  for (int step = wk; step < full; step += WK) {
    turn([&] {
#pragma unroll
      for (int i = 0; i < S::kBlocks; ++i) load(i, step + WK < full ? step + WK : step);
    });
    multiply();
  }

  const TensorScales ts{A.ts, B.ts, A.ts_per_row != 0, B.ts_per_row != 0};
  const bool vec = ts.a_per_row || ts.b_per_row;
  const float out_scale = vec ? 0.0f : A.ts[0] * B.ts[0];
  auto store = [&](float4v v, int i, int j) {
    const int m = m0 + i * 16 + l16, n = n0 + j * 16 + q * 4;
    if (m < M && n < N) {
      v *= scale4(ts, out_scale, vec, true, m, n);
      if (kBf16Out) {
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

}  // namespace

// The tile shapes the kernel comes in.  In the first four the wavefronts of a workgroup split K.  Which of these: `cost` is the time
// of one step (128 k) of one round of 256 tiles, in units of 0.247 us, fitted to the measured times of 13 shapes (it reproduces them
// within 5 %); a shape's time is then
//   3 us + 0.247 us * cost * steps * ceil(tiles / 256),
// and the smallest wins: large tiles decode less per product, small ones fill the chip.  Both sides of the choice, us:
// 64 x 20480 x 5120: 4x3 22.3, 4x4 26.7, 2x2 27.2; 512 x 5120 x 5120: 4x4 37.8, 4x3 39.4; 32 x 5120 x 5120: 2x2 7.7, 1x2 8.8, 4x3 > 10.
// The last has a tile per wavefront, 128 x 128 outputs per workgroup: for results that fill the chip without a split of K, where the
// others' wavefronts have too few steps to share and pay the sum through LDS per 64 x 64 tile.  Which of the two: `us`, fitted to
// 930 measured calls of 16 .. 8192 rows, 256 .. 20480 columns, K 16 .. 20496, FP32 and bf16 (its 5th and 95th percentile are 0.85 and 1.12
// of the measured time).  us, 4x4 split / own: 5120 x 20480 x 16 193 / 87, x 400 228 / 159, x 2064 677 / 623; 2048 x 5120 x 2064 the split.
struct DirectShape {
  int mb, nb, wk;
  double cost;
  SmallTileCost us;
};
constexpr DirectShape kDirectShapes[5] = {{1, 2, 8, 0.30, {3, 4.02, 1.23, 0.0, 0.647, 0.203}},
                                          {2, 2, 8, 0.46, {2, 3.53, 1.0, 0.0, 1.02, 0.214}},
                                          {4, 3, 4, 0.96, {2, 4.01, 1.15, 0.591, 0.936, 0.194}},
                                          {4, 4, 4, 1.19, {2, 4.09, 1.03, 0.653, 1.17, 0.186}},
                                          {4, 4, 1, 0.0, {2, 3.72, 1.13, 1.56, 1.14, 0.141}}};

// (Shapes as template arguments: every division is by a constant.)
template <int I>
static int64_t direct_tiles(int64_t M, int64_t N) {
  constexpr DirectShape d = kDirectShapes[I];
  constexpr int tm = d.mb * (d.wk == 1 ? 32 : 16), tn = d.nb * (d.wk == 1 ? 32 : 16);
  return ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
}

// What the kernel's 32-bit rows, byte offsets within a 16-row block and launch size allow; others take other kernels.
template <int I>
static bool fits(int64_t M, int64_t N, int64_t K) {
  constexpr int wk = kDirectShapes[I].wk;
  return M <= 0x7fffffff && N <= 0x7fffffff && K <= (int64_t{1} << 27) && direct_tiles<I>(M, N) * (wk == 1 ? 256 : wk * 64) <= 0xffffffff;
}

template <int I>
static void consider(int64_t M, int64_t N, int64_t K, DirectPick& best) {
  if (!fits<I>(M, N, K)) return;
  const int64_t tiles = direct_tiles<I>(M, N), rounds = (tiles + 255) / 256, steps = (K + kStepK - 1) / kStepK;
  const double us = 3.0 + 0.247 * kDirectShapes[I].cost * static_cast<double>(steps) * static_cast<double>(rounds);
  if (us < best.compute_us) best = DirectPick{I, tiles, us};
}

DirectPick pick_direct_shape(const GemmArgs& g) {
  DirectPick best{0, 0, HUGE_VAL};
  consider<0>(g.a.outer, g.b.outer, g.K, best);
  consider<1>(g.a.outer, g.b.outer, g.K, best);
  consider<2>(g.a.outer, g.b.outer, g.K, best);
  consider<3>(g.a.outer, g.b.outer, g.K, best);
  return best;
}

template <int I>
static double shape_us(const GemmArgs& g) {
  if (!fits<I>(g.a.outer, g.b.outer, g.K)) return HUGE_VAL;
  constexpr DirectShape d = kDirectShapes[I];
  const int64_t steps = (g.K + kStepK - 1) / kStepK;
  return small_tile_us(d.us, direct_tiles<I>(g.a.outer, g.b.outer), static_cast<double>(g.a.outer) * static_cast<double>(g.b.outer),
                       (steps + d.wk - 1) / d.wk);
}

double gemm_direct_us(const GemmArgs& g, int shape) {
  switch (shape) {
    case 0: return shape_us<0>(g);
    case 1: return shape_us<1>(g);
    case 2: return shape_us<2>(g);
    case 3: return shape_us<3>(g);
    default: return shape_us<kDirectOwnTiles>(g);
  }
}

template <int MB, int NB, int WK, bool kBf16Out>
static hipError_t launch_shape(const GemmArgs& g, hipStream_t s) {
  using S = Shape<MB, NB, WK>;
  static PerDeviceOnce once;
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_direct_kernel<MB, NB, WK, kBf16Out>), S::kLdsBytes, once);
  if (e != hipSuccess) return e;
  const int tiles_m = static_cast<int>((g.a.outer + S::kTM - 1) / S::kTM), tiles_n = static_cast<int>((g.b.outer + S::kTN - 1) / S::kTN);
  hipLaunchKernelGGL((gemm_direct_kernel<MB, NB, WK, kBf16Out>), dim3(static_cast<unsigned>(tiles_m * tiles_n)), dim3(S::kThreads),
                     S::kLdsBytes, s, g.a, g.b, static_cast<int>(g.K), g.d, g.ldd, g.accumulate, tiles_m, tiles_n);
  return hipGetLastError();
}

template <bool kBf16Out>
static hipError_t launch_direct(const GemmArgs& g, int shape, hipStream_t s) {
  switch (shape) {
    // 16 x 32 tiles: enough of them to fill the chip four times over do better with fewer wavefronts on each (16 x 20480 x
    // 5120: 14.6 against 15.7 us), few with more (32 x 5120 x 5120 in these tiles: 9.4 against 8.8)
    case 0: return direct_tiles<0>(g.a.outer, g.b.outer) >= 512 ? launch_shape<1, 2, 4, kBf16Out>(g, s) : launch_shape<1, 2, 8, kBf16Out>(g, s);
    case 1: return launch_shape<2, 2, 8, kBf16Out>(g, s);
    case 2: return launch_shape<4, 3, 4, kBf16Out>(g, s);
    case 3: return launch_shape<4, 4, 4, kBf16Out>(g, s);
    default: return launch_shape<4, 4, 1, kBf16Out>(g, s);
  }
}

hipError_t launch_gemm_direct(const GemmArgs& g, int shape, hipStream_t s) {
  if (gemm_direct_us(g, shape) == HUGE_VAL) return hipErrorInvalidValue;   // beyond its offsets or a launch
  return g.out_bf16 ? launch_direct<true>(g, shape, s) : launch_direct<false>(g, shape, s);
}

}  // namespace nvfp4
