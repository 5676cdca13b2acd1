// MXFP4 GEMM for gfx950 on the block-scaled matrix instruction: the paper's
// comparison format (Sec. 2: E2M1 elements, one UE8M0 power-of-two scale per 32)
// is exactly what v_mfma_scale_f32_16x16x128_f8f6f4 consumes, so -- unlike the
// NVFP4 GEMM, whose E4M3-per-16 scales force a decode to FP16 -- the packed codes
// go from global memory through LDS into the matrix pipe untouched:
//   D[m, n] = sum_b 2^(ea[m,b] + eb[n,b]) sum_{k in b} A[m,k] B[n,k],  FP32 accumulation.
//
// Operand layout of the instruction with FP4 inputs (checked on the device):
// lane l carries row (l & 15) and the 32 consecutive k of block (l >> 4) as 16
// bytes (element 2t in the low nibble of byte t -- the storage format as it is)
// plus that block's scale byte; the 16x16 result puts D[(l >> 4) * 4 + i][l & 15]
// in register i of lane l, rows taken from the first operand.
//
// The kernel for any K: 256 x 256 outputs per workgroup, K step 128 (one instruction deep), 256 threads = 4 wavefronts
// (2 x 2), one per SIMD, of 128 x 128 outputs each: 8 x 8 instructions per K step, 256 accumulator
// registers in the accumulation half of the register file.  LDS holds two buffers of two K steps,
// a step being (A codes, B codes, A scales, B scales) = 34 KiB, filled by direct global->LDS
// loads: a code row of a step is 64 bytes, so 16 consecutive tile rows are 1 KiB of LDS and a
// fragment read (16 rows x 4 blocks x 16 bytes) is one contiguous KiB.
//
// With one wavefront per SIMD nothing else can fill the matrix pipe while this one waits, so the
// loop is software-pipelined across its barrier and its instruction order is fixed by hand (inline
// assembly; the compiler would regroup it).  One iteration = the two K steps of a buffer:
//   block 1   64 MFMAs on the first step; behind them the 24 fragment reads of the second
//   wait      own reads back, own global->LDS loads (issued one iteration ago) landed; barrier:
//             every wavefront holds all it needs of this buffer, and the other buffer is complete
//   block 2   64 MFMAs on the second step; behind them the reads for the first step of the
//             other buffer and the 20 loads that refill this one with the steps after that
#include <type_traits>

#include "nvfp4_internal.h"
#include "nvfp4_device.h"
#include "gemm_epilogue.h"

namespace nvfp4 {

namespace {

constexpr int TM = 256, TN = 256, TK = 128;
constexpr int kThreads = 256;
constexpr int kCodeRowBytes = TK / 2;                 // 64
constexpr int kCodeBytes = TM * kCodeRowBytes;        // 16 KiB per operand
constexpr int kScaleBytes = TM * (TK / 32);           // 1 KiB per operand
constexpr int kStepBytes = 2 * kCodeBytes + 2 * kScaleBytes;   // 34 KiB
constexpr int kLdsBytes = 4 * kStepBytes;

typedef int int4v __attribute__((ext_vector_type(4)));

template <int kBegin, int kEnd, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kBegin < kEnd) {
    f(std::integral_constant<int, kBegin>{});
    static_for<kBegin + 1, kEnd>(f);
  }
}

// 64 lanes x 16 (or 4) bytes from global memory (wave-uniform base + per-lane 32-bit offset) straight
// into consecutive LDS at the wave-uniform LDS address lds_dst (M0 carries it).  Asynchronous (vmcnt).
__device__ __forceinline__ void load16_to_lds(uint32_t lane_offset, const uint8_t* base, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_dst), "v"(lane_offset), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void load4_to_lds(uint32_t lane_offset, const uint8_t* base, uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_dst), "v"(lane_offset), "s"(base)
               : "memory", "m0");
}

// The same kOff bytes on: the instruction's immediate offset is added to the LDS address and to the global address alike, so the
// caller passes a global address that is kOff too low.  M0 is an operand: where a following load has the same lds_dst the compiler sets it once for
// both, and whatever else it may put into M0 in between it undoes.  (s_nop: the wait state that M0 needs when it has just been set.)
template <int kOff>
__device__ __forceinline__ void load16_to_lds_at(uint32_t lane_offset, const uint8_t* base, uint32_t lds_dst) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(lane_offset), "s"(base), "n"(kOff), "{m0}"(lds_dst) : "memory");
}

// LDS reads; asynchronous, the caller waits (lgkmcnt) before the values are used.
template <int kOff>
__device__ __forceinline__ void lds_read16(int4v& dst, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(dst) : "v"(addr), "n"(kOff));
}
typedef int int2v __attribute__((ext_vector_type(2)));
// two dwords, kOff0 and kOff1 dwords past addr
template <int kOff0, int kOff1>
__device__ __forceinline__ void lds_read_2x4(int2v& dst, uint32_t addr) {
  asm volatile("ds_read2_b32 %0, %1 offset0:%2 offset1:%3" : "=&v"(dst) : "v"(addr), "n"(kOff0), "n"(kOff1));
}
// byte k of the result = byte sel[k] of the eight bytes {hi, lo}; in assembly so that it stays behind the
// wait for the LDS reads that produce its inputs (the compiler does not know those are asynchronous)
__device__ __forceinline__ int perm_bytes(int hi, int lo, int sel) {
  int d;
  asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(d) : "v"(hi), "v"(lo), "v"(sel));
  return d;
}

// Fragments of one K step for a 128 x 128 wave tile: per 16-row block the lane's 32 codes (the
// instruction's FP4 operand is four dwords) and its block's scale byte.  Single-byte LDS reads are slow
// (measured: 16 of them per K step cost more than the 64 MFMAs), so the scales are read as the row's whole
// dword (the step's four blocks) and the lane's own byte of four rows is gathered into one register (pa, pb);
// the instruction then picks the row's byte with its op_sel field.
constexpr int kFragReads = 24;
struct Frags {
  int4v a[8], b[8];
  int pa[2], pb[2];     // byte t of pa[h] = this lane's scale of block 4h + t
};
// Raw scale dwords of 16-row blocks (2t, 2t + 1) between their read and the gather; one set serves both
// fragment sets, whose reads never overlap (each set is gathered before the other's reads start).
struct RawScales {
  int2v a[4], b[4];
};

// Read number q of the 24 of a fragment set: 0..7 A codes, 8..15 B codes, 16..19 A scales, 20..23 B scales
// (16-row blocks are 1 KiB of codes and 64 bytes = 16 dwords of scales apart).
template <int q>
__device__ __forceinline__ void read_frag(Frags& f, RawScales& r, uint32_t a_codes, uint32_t b_codes, uint32_t a_scales,
                                          uint32_t b_scales) {
  if constexpr (q < 8) lds_read16<q * 16 * kCodeRowBytes>(f.a[q], a_codes);
  else if constexpr (q < 16) lds_read16<(q - 8) * 16 * kCodeRowBytes>(f.b[q - 8], b_codes);
  else if constexpr (q < 20) lds_read_2x4<(q - 16) * 32, (q - 16) * 32 + 16>(r.a[q - 16], a_scales);
  else lds_read_2x4<(q - 20) * 32, (q - 20) * 32 + 16>(r.b[q - 20], b_scales);
}

// After the reads are back: gather the lane's byte (sel01 = kb | (4 + kb) << 8 picks byte kb of two dwords).
__device__ __forceinline__ void pack_scales(Frags& f, const RawScales& r, int sel01) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int a01 = perm_bytes(r.a[2 * h][1], r.a[2 * h][0], sel01), a23 = perm_bytes(r.a[2 * h + 1][1], r.a[2 * h + 1][0], sel01);
    f.pa[h] = perm_bytes(a23, a01, 0x05040100);
    const int b01 = perm_bytes(r.b[2 * h][1], r.b[2 * h][0], sel01), b23 = perm_bytes(r.b[2 * h + 1][1], r.b[2 * h + 1][0], sel01);
    f.pb[h] = perm_bytes(b23, b01, 0x05040100);
  }
}

// The instruction's first operand supplies the rows of its result: passing B first leaves a lane with 4
// consecutive n of one m, which makes the output stores 64/128-bit.  cbsz / blgp = 4: both operands FP4;
// scale byte kSelB of sb and kSelA of sa (op_sel = the low bit, op_sel_hi = the high bit of the byte number).
// The accumulator is pinned to the accumulation registers.
template <int kSelB, int kSelA>
__device__ __forceinline__ void mfma(float4v& acc, const int4v& b, const int4v& a, int sb, int sa) {
  asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel:[%5,%6,0] op_sel_hi:[%7,%8,0] cbsz:4 blgp:4"
               : "+a"(acc)
               : "v"(b), "v"(a), "v"(sb), "v"(sa), "n"(kSelB & 1), "n"(kSelA & 1), "n"(kSelB >> 1), "n"(kSelA >> 1));
}

// For K not a multiple of 512, and scales that are not 16-byte aligned.  Bound by the number of line requests (see gemm_mx_kernel_k512): 4096 x 5120 with K = 4224, 4352, 4480 takes 94, 93, 100 us
// (bf16; FP32 102, 102, 108), where the other kernel takes 47 and 48 (49, 53) with K = 4096 and 4608; with K = 128 and 640 19 and 28 (27, 35).
template <bool kBf16Out>
__global__ __launch_bounds__(kThreads) void gemm_mx_kernel_any_k(Operand A, Operand B, int64_t K, void* __restrict__ Dv,
                                                                 int64_t ldd, bool accumulate, int tiles_m, int tiles_n) {
  extern __shared__ __attribute__((aligned(16))) char lds[];

  // Workgroup -> tile: consecutive ids go to different XCDs (round robin over 8, one L2 each);
  // every XCD gets a contiguous range of tiles, walked in bands of 8 tile rows.
  const int num_tiles = tiles_m * tiles_n;
  int pid = blockIdx.x;
  if ((num_tiles & 7) == 0) pid = (pid & 7) * (num_tiles >> 3) + (pid >> 3);
  constexpr int kBand = 8;
  const int band = pid / (kBand * tiles_n);
  const int band_rows = min(kBand, tiles_m - band * kBand);
  const int in_band = pid - band * kBand * tiles_n;
  const int tm = band * kBand + in_band % band_rows, tn = in_band / band_rows;
  const int64_t m0 = static_cast<int64_t>(tm) * TM, n0 = static_cast<int64_t>(tn) * TN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, kb = lane >> 4;
  const int arow = wm * 128 + l16, brow = wn * 128 + l16;
  const int64_t code_ld = K / 2, scale_ld = K / 32;

  // Direct-load sources = wave-uniform 64-bit base + per-lane 32-bit offset.  Codes: an instruction fills 16 tile
  // rows (lane -> row lane / 4, 16-byte piece lane % 4), so one per-lane offset serves every instruction and both
  // operands (a 16-row block is at most 16 * K / 2 bytes: K < 2^24, checked on the host); every wavefront loads 64
  // rows of A and of B.  A 16-row block past the end of an operand is replaced by the operand's last block (rows
  // come in multiples of 32, so a block is in or out as a whole); it only feeds outputs that are never stored.
  // Scales: an instruction fills 64 tile rows x 4 bytes, rows clamped per lane; every wavefront loads its 64 rows.
  const uint32_t off_codes = static_cast<uint32_t>(lane >> 2) * static_cast<uint32_t>(code_ld) + (lane & 3) * 16;
  const uint32_t off_sa = static_cast<uint32_t>(min<int64_t>(wave * 64 + lane, A.outer - 1 - m0)) * static_cast<uint32_t>(scale_ld);
  const uint32_t off_sb = static_cast<uint32_t>(min<int64_t>(wave * 64 + lane, B.outer - 1 - n0)) * static_cast<uint32_t>(scale_ld);
  const uint8_t* tile_sa = A.scales + m0 * scale_ld;
  const uint8_t* tile_sb = B.scales + n0 * scale_ld;
  const uint8_t* blk_a[4];
  const uint8_t* blk_b[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t r = (wave * 4 + q) * 16;
    blk_a[q] = A.codes + (m0 + min<int64_t>(r, A.outer - 16 - m0)) * code_ld;
    blk_b[q] = B.codes + (n0 + min<int64_t>(r, B.outer - 16 - n0)) * code_ld;
  }
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  // load number q (0..9) of K step kt into step slot `slot` (0..3): 0..3 A codes, 4..7 B codes, 8 A scales, 9 B scales
  auto issue_one = [&](int q, int kt, int slot) {
    const uint32_t base = lds0 + slot * kStepBytes;
    if (q < 4)
      load16_to_lds(off_codes, blk_a[q & 3] + static_cast<int64_t>(kt) * kCodeRowBytes, base + (wave * 4 + q) * 1024);
    else if (q < 8)
      load16_to_lds(off_codes, blk_b[q & 3] + static_cast<int64_t>(kt) * kCodeRowBytes, base + kCodeBytes + (wave * 4 + (q & 3)) * 1024);
    else if (q == 8)
      load4_to_lds(off_sa, tile_sa + static_cast<int64_t>(kt) * 4, base + 2 * kCodeBytes + wave * 256);
    else
      load4_to_lds(off_sb, tile_sb + static_cast<int64_t>(kt) * 4, base + 2 * kCodeBytes + kScaleBytes + wave * 256);
  };
  // fragment addresses in step slot 0
  const uint32_t a_codes = lds0 + arow * kCodeRowBytes + kb * 16, b_codes = lds0 + kCodeBytes + brow * kCodeRowBytes + kb * 16;
  const uint32_t a_scales = lds0 + 2 * kCodeBytes + arow * 4, b_scales = lds0 + 2 * kCodeBytes + kScaleBytes + brow * 4;
  const int sel01 = kb | ((4 + kb) << 8);

  float4v acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

  const int KT = static_cast<int>(K / TK);
  // K steps 0..3 into step slots 0..3.  Steps past the end are clamped to the last one: they land in slots nobody
  // multiplies any more, and no branch is needed.
  static_for<0, 40>([&](auto ic) {
    constexpr int n = decltype(ic)::value;
    issue_one(n % 10, min(n / 10, KT - 1), n / 10);
  });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  Frags f0, f1;
  RawScales raw;
  static_for<0, kFragReads>([&](auto q) { read_frag<decltype(q)::value>(f0, raw, a_codes, b_codes, a_scales, b_scales); });
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  pack_scales(f0, raw, sel01);

  for (int kt = 0; kt < KT; kt += 2) {
    const uint32_t cur = ((kt >> 1) & 1) * (2 * kStepBytes), nxt = cur ^ (2 * kStepBytes);
    const uint32_t second = cur + kStepBytes;
    static_for<0, 64>([&](auto ic) {
      constexpr int n = decltype(ic)::value;
      mfma<(n & 3), ((n >> 3) & 3)>(acc[n >> 3][n & 7], f0.b[n & 7], f0.a[n >> 3], f0.pb[(n & 7) >> 2], f0.pa[n >> 5]);
      if constexpr ((n & 1) == 1 && (n >> 1) < kFragReads)
        read_frag<(n >> 1)>(f1, raw, a_codes + second, b_codes + second, a_scales + second, b_scales + second);
    });
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    pack_scales(f1, raw, sel01);
    if (kt + 1 < KT) {   // an odd number of K steps leaves the last buffer's second step empty
      const int slot = ((kt >> 1) & 1) * 2;
      const int kt4 = min(kt + 4, KT - 1), kt5 = min(kt + 5, KT - 1);
      static_for<0, 64>([&](auto ic) {
        constexpr int n = decltype(ic)::value;
        mfma<(n & 3), ((n >> 3) & 3)>(acc[n >> 3][n & 7], f1.b[n & 7], f1.a[n >> 3], f1.pb[(n & 7) >> 2], f1.pa[n >> 5]);
        if constexpr ((n & 1) == 0 && (n >> 1) < kFragReads)
          read_frag<(n >> 1)>(f0, raw, a_codes + nxt, b_codes + nxt, a_scales + nxt, b_scales + nxt);
        if constexpr ((n & 1) == 1 && n < 40)
          issue_one((n >> 1) % 10, (n >> 1) < 10 ? kt4 : kt5, slot + ((n >> 1) < 10 ? 0 : 1));
      });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      pack_scales(f0, raw, sel01);
    }
  }
  // The trailing global->LDS loads must have landed before the wavefront ends; the MFMA results must have left
  // the pipe before ordinary instructions read the accumulators (the compiler cannot see into the assembly
  // statements to insert these wait states itself).
  asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");

  const TensorScales out_scale{A.ts, B.ts, false, false};    // both are 1 for MXFP4 (no tensor-level scale)
  const int Mt = static_cast<int>(A.outer - m0 < TM ? A.outer - m0 : TM);
  const int Nt = static_cast<int>(B.outer - n0 < TN ? B.outer - n0 : TN);
  store_wave_block<kBf16Out>(acc, out_scale, Dv, ldd, accumulate, m0 + wm * 128, n0 + wn * 128, Mt - wm * 128, Nt - wn * 128,
                             lane);
}

// ---------------------------------------------------------------- K a multiple of 512
// The kernel above asks the memory system for many small pieces: per K step a 64-byte piece of every code row
// and a 4-byte piece of every scale row, each its own cache-line request (measured: about one request per
// clock and CU, which is what bounds it).  When K is a multiple of 512 this one runs on fuller lines:
//   codes   a stage is two K steps = 128 bytes of each row, 8 rows per load instruction, stored with the XOR
//           swizzle chunk c of row r -> position c ^ ((r >> 1) & 7) so that fragment reads stay conflict-free;
//           the two steps of a stage are the two 64-byte halves of its rows
//   scales  16 bytes of each scale row = four K steps = two stages per load instruction; a wavefront reads 64 rows' 16 bytes at once and transposes them
//           between its lanes, a step's while the step before runs (behind its MFMAs: bunched between two steps 20 of these instructions cost 90 cycles)
// a third of the line requests for the same bytes.  What bounds it is loading: a CU takes in 64 bytes a clock, which for 256 x 160 tiles is two thirds of the time that
// the MFMAs on them take, for 256 x 320 less than half.  So the loop keeps one set of fragments, which leaves room for 128 x 160 outputs per wavefront (320 accumulators): a
// step runs the upper half of the wavefront's blocks column by column, then the lower half, and a fragment's registers take its next values once its last MFMA
// has been issued.  The stage's last reads are those of the second step's lower A fragments, at the start of it; the loads that refill the buffer go
// behind the rest of that step, and have landed in the middle of the next stage's second step.
// us per call, two sets of fragments in tiles of up to 256 columns -> now: 4096 x 5120 x 5120 bf16 62.8 -> 53.1 (256 x 320; 256 x 160 60.4), 5120 x 5120 x 4096 FP32 69.3 -> 68.2
// (256 x 224), 8192 x 20480 x 5120 bf16 431 -> 401 (4.3 PFLOP/s), 2048 x 5120 x 5120 33.5 -> 32.2.  Over 120 products of 0.3 to 170 million outputs 4 % less time.
constexpr int kWideRowBytes = 128;
constexpr int wide_stage_bytes(int nb) { return (TM + 32 * nb) * kWideRowBytes; }
constexpr int wide_lds_bytes(int nb) { return 2 * wide_stage_bytes(nb) + (TM + 32 * nb) * 16 + 768; }   // two stages, one chunk of scales (read in whole KiBs: up to 48 rows past the end)

__device__ __forceinline__ int swz128(int row, int chunk) { return row * kWideRowBytes + ((chunk ^ ((row >> 1) & 7)) << 4); }

// Byte t of the result = this lane's scale (block l >> 4 of the step) of 16-row block 4 h + t: a 4 x 4 transposition of bytes over the four lanes that
// hold a row number's dwords: half-wavefronts exchanged and two bytes of each kept, then 16-lane rows and one byte of each.
__device__ __forceinline__ uint32_t transpose_half(int v, uint32_t sel_half) {
  const auto h = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(v), static_cast<uint32_t>(v), false, false);
  return __builtin_amdgcn_perm(h[1], h[0], sel_half);
}
__device__ __forceinline__ int transpose_row(uint32_t u, uint32_t sel_row) {
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return static_cast<int>(__builtin_amdgcn_perm(r[1], r[0], sel_row));
}

// 16 bytes of LDS at addr + kOff, kNew: into any registers; else into those that the fragment has (an operand in and out).
template <int kOff, bool kNew>
__device__ __forceinline__ void lds_read_frag(int4v& dst, uint32_t addr) {
  if constexpr (kNew) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(dst) : "v"(addr), "n"(kOff));
  else asm volatile("ds_read_b128 %0, %1 offset:%2" : "+v"(dst) : "v"(addr), "n"(kOff));
}
// No instruction: the value is used here / comes from here.
__device__ __forceinline__ void keep(const int4v& f) { asm volatile("" ::"v"(f)); }
__device__ __forceinline__ void arrived(int4v& f) { asm volatile("" : "+v"(f)); }
__device__ __forceinline__ void turned(int& scale) { asm volatile("" : "+v"(scale)); }   // what makes it stays ahead of the statements behind this, what uses it behind it
template <bool kAcc>
__device__ __forceinline__ void settled(float4v& acc) {
  if constexpr (kAcc) asm volatile("" : "+a"(acc));
  else asm volatile("" : "+v"(acc));
}

// The instruction as above; kAcc: accumulator in the accumulation registers; kFirst: the first on an accumulator in a tile, C = 0, so they are never cleared.
template <bool kFirst, bool kAcc, int kSelB, int kSelA>
__device__ __forceinline__ void mfma_wide(float4v& acc, const int4v& b, const int4v& a, int sb, int sa) {
#define NVFP4_MFMA_MX(DST, C)                                                                                                          \
  asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, " C ", %3, %4 op_sel:[%5,%6,0] op_sel_hi:[%7,%8,0] cbsz:4 blgp:4"        \
               : DST(acc)                                                                                                              \
               : "v"(b), "v"(a), "v"(sb), "v"(sa), "n"(kSelB & 1), "n"(kSelA & 1), "n"(kSelB >> 1), "n"(kSelA >> 1))
  if constexpr (kFirst && kAcc) NVFP4_MFMA_MX("=a", "0");
  else if constexpr (kFirst) NVFP4_MFMA_MX("=v", "0");
  else if constexpr (kAcc) NVFP4_MFMA_MX("+a", "%0");
  else NVFP4_MFMA_MX("+v", "%0");
#undef NVFP4_MFMA_MX
}

// A wavefront's output stage issues 8 ceil(kNB / 2) (bf16) or 8 kNB (FP32) stores for a full tile; three quarters of them may still be
// outstanding when the loads issued before it are needed (memory operations complete in issue order).
template <bool kBf16Out, int kNB>
constexpr int kTileStoresMx = 6 * (kBf16Out ? (kNB + 1) / 2 : kNB);

// What goes behind the MFMAs of a K step.  kR rows of blocks a half; MFMA n of a half is in column n / kR.
template <int kNB>
struct Schedule {
  static constexpr int kMB = 8, kR = kMB / 2, kHalf = kR * kNB;
  static constexpr int kLoads = kMB + kNB;            // a wavefront's code loads per stage
  static constexpr int kA = kMB / 4, kB = (kNB + 3) / 4;   // registers of packed scales; reads of a chunk's scales
  static constexpr int kFree = kR + 6 < kHalf - 4 ? kR + 6 : kHalf - 4;   // in the upper half of a stage's second step: before it everybody has read the stage out
  static constexpr int kLoadPlaces = 2 * kHalf - kFree;
  static constexpr int spread(int n, int total, int slots) { return (n + 1) * total / slots > n * total / slots ? n * total / slots : -1; }
  static constexpr int load(int n) { return spread(n, kLoads, kLoadPlaces); }   // n counts from kFree on
  static constexpr int kEarlyLoads = (kHalf - kFree) * kLoads / kLoadPlaces;    // of them in the upper half
  // upper half: which A fragment of the lower half is read behind MFMA n (at once: the stage's second step frees the buffer then)
  static constexpr int upper_read(int n) { return n >= 1 && n <= kR ? kR + n - 1 : -1; }
  static constexpr int upper_reads_before(int n) { return n <= 1 ? 0 : n - 1 < kR ? n - 1 : kR; }
  // lower half: which upper A fragment of the next step (all of them before the last two of B), and which B fragment
  static constexpr int kGapA = 2 + kR * (kR - 1) < kR * (kNB - 2) ? kR : 2 + 3 * (kR - 1) < kR * (kNB - 2) ? 3 : 1;
  static_assert(2 + kGapA * (kR - 1) < kR * (kNB - 2), "the last two reads of a step are of B");
  static constexpr int lower_read_a(int n) { return n >= 2 && (n - 2) % kGapA == 0 && (n - 2) / kGapA < kR ? (n - 2) / kGapA : -1; }
  static constexpr int lower_read_b(int n) { return n >= kR && n % kR == 0 ? n / kR - 1 : -1; }   // (the last column's: behind the next step's first MFMA)
  static constexpr int lower_reads_behind_a() {   // of B
    int r = 0;
    for (int k = 2 + kGapA * (kR - 1); k < kHalf; ++k) r += lower_read_b(k) >= 0;
    return r;
  }
  static constexpr int lower_reads_before(int n) {
    int r = 0;
    for (int k = 0; k < n; ++k) r += (lower_read_a(k) >= 0) + (lower_read_b(k) >= 0);
    return r;
  }
  // lower half: the next step's scales are turned in 2 (kA + kB) pieces, one behind each of some MFMAs of the second half of it but the last: an MFMA may read a
  // vector instruction's result two instructions later at the earliest, and the compiler sees no MFMA in the statements that it could keep apart
  static constexpr int kTurnFrom = kHalf / 2, kTurnPlaces = kHalf - kTurnFrom - 1;
  static constexpr int turn(int n) { return n >= kTurnFrom && n < kHalf - 1 ? spread(n - kTurnFrom, 2 * (kA + kB), kTurnPlaces) : -1; }
  static_assert(2 * (kA + kB) <= kTurnPlaces, "a piece of the turn behind each MFMA at the most");
};

// With more tiles than CUs the host launches one workgroup per CU, which takes tiles blockIdx.x, blockIdx.x +
// gridDim.x, ... and runs them as ONE stream of stages, as the FP16 kernel of the NVFP4 route does: the loads issued
// during a tile's last two stages fetch the next tile's first two (and its first scale chunk), so the pipeline
// neither drains nor refills at a tile boundary.  K is a multiple of 512, so every tile is an even number of stages
// and a whole number of scale chunks: the stage buffers simply keep turning.  The output stage's stores are not waited for.
// kNB: 16-column blocks per wavefront (2 x 2 wavefronts of 8 16-row blocks).
template <bool kBf16Out, int kNB>
__global__ __launch_bounds__(kThreads) void gemm_mx_kernel_k512(Operand A, Operand B, int64_t K, void* __restrict__ Dv,
                                                                int64_t ldd, bool accumulate, int tiles_m, int tiles_n) {
  using S = Schedule<kNB>;
  constexpr int kMB = S::kMB, kTM = TM, kTN = 32 * kNB, kStageBytes = wide_stage_bytes(kNB), kOperandBytes = kTM * kWideRowBytes;
  constexpr int kR = S::kR, kHalf = S::kHalf;
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int num_tiles = tiles_m * tiles_n;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int64_t code_ld = K / 2, scale_ld = K / 32;
  // Work item -> tile: consecutive workgroup ids go to different XCDs (round robin over 8, one L2 each); every XCD
  // gets a contiguous range of tiles, walked in bands of 8 tile rows.
  auto locate = [&](int item, int& tm, int& tn) {
    if ((num_tiles & 7) == 0) item = (item & 7) * (num_tiles >> 3) + (item >> 3);
    tile_coordinates(item, tiles_m, tiles_n, tm, tn);
  };

  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const uint32_t scales0 = lds0 + 2 * kStageBytes;
  // What depends on the lane is worked out once per tile, from a lane number asked for on the spot (values kept from
  // before the first tile would have to live through every output stage and end up in scratch memory).
  // Code loads: instruction q of wavefront w fills 8 rows of a tile, rows 8 (w kMB + q) of A's, 8 (w kNB + q) of B's (lane -> row lane / 8,
  // position lane % 8, i.e. chunk (lane % 8) ^ ((row >> 1) & 7), which an odd 8-row block flips bit 2 of).  Scale loads: one instruction = 64 tile rows x 16 bytes (four K steps).
  uint32_t lane_even = 0, lane_odd = 0, lane_srow = 0;
  uint32_t a_lo = 0, a_hi = 0, b_lo = 0, b_hi = 0, a_scales = 0, b_scales = 0;   // fragment addresses: stage buffer 0, step 0 / 1
  uint32_t sel_half = 0, sel_row = 0;   // of the turn of the scales
  auto lane_setup = [&]() {
    const int lane = lane_id();
    const uint32_t c0 = static_cast<uint32_t>((lane & 7) ^ ((lane >> 4) & 7)) * 16u;
    lane_even = static_cast<uint32_t>(lane >> 3) * static_cast<uint32_t>(code_ld) + c0;
    lane_odd = static_cast<uint32_t>(lane >> 3) * static_cast<uint32_t>(code_ld) + (c0 ^ 64u);
    lane_srow = static_cast<uint32_t>(lane);
    const int l16 = lane & 15, kb = lane >> 4;
    const int arow = (wave >> 1) * (16 * kMB) + l16, brow = (wave & 1) * (16 * kNB) + l16;
    a_lo = lds0 + swz128(arow, kb);
    a_hi = lds0 + swz128(arow, 4 + kb);
    b_lo = lds0 + kOperandBytes + swz128(brow, kb);
    b_hi = lds0 + kOperandBytes + swz128(brow, 4 + kb);
    a_scales = scales0 + ((wave >> 1) * (16 * kMB) + lane) * 16;
    b_scales = scales0 + kTM * 16 + ((wave & 1) * (16 * kNB) + lane) * 16;
    sel_half = kb < 2 ? 0x05040100u : 0x07060302u;
    sel_row = (kb & 1) == 0 ? 0x06020400u : 0x07030501u;
  };
  lane_setup();
  // Load addresses: a wave-uniform 64-bit base per operand (codes, scales), which holds the tile and the stage /
  // scale chunk being fetched, plus per-lane 32-bit offsets, which hold the row and the chunk and do not change
  // within a tile (320 rows of K / 2 bytes: K < 2^24, checked on the host): moving the loads on is scalar work.  An 8-row block past the end of an operand is replaced by the operand's last block (rows come in
  // multiples of 32); it only feeds outputs that are never stored.  Scale rows are clamped per lane.
  const uint8_t* base_a = nullptr;
  const uint8_t* base_b = nullptr;
  const uint8_t* base_sa = nullptr;
  const uint8_t* base_sb = nullptr;
  uint32_t last_a = 0, last_b = 0;   // rows that a load of 8 may start at the most
  uint32_t voff[kMB + kNB];          // A's, then B's
  // Point the loads at stage `stage` and scale chunk `chunk` of tile (tm, tn).
  auto aim = [&](int tm, int tn, int stage, int chunk) {
    const int64_t m_first = static_cast<int64_t>(tm) * kTM, n_first = static_cast<int64_t>(tn) * kTN;
    base_a = A.codes + m_first * code_ld + stage * kWideRowBytes - 3072;
    base_b = B.codes + n_first * code_ld + stage * kWideRowBytes - 3072;
    base_sa = A.scales + m_first * scale_ld + chunk * 16;
    base_sb = B.scales + n_first * scale_ld + chunk * 16;
    last_a = static_cast<uint32_t>(A.outer - 8 - m_first), last_b = static_cast<uint32_t>(B.outer - 8 - n_first);
#pragma unroll
    for (int q = 0; q < kMB; ++q) {
      const uint32_t blk = static_cast<uint32_t>(wave * kMB + q);
      voff[q] = ((blk & 1) ? lane_odd : lane_even) + min(blk * 8u, last_a) * static_cast<uint32_t>(code_ld) + (3 - (q & 3)) * 1024u;
    }
#pragma unroll
    for (int q = 0; q < kNB; ++q) {
      const uint32_t blk = static_cast<uint32_t>(wave * kNB + q);
      voff[kMB + q] = ((blk & 1) ? lane_odd : lane_even) + min(blk * 8u, last_b) * static_cast<uint32_t>(code_ld) + (3 - (q & 3)) * 1024u;
    }
  };
  // Load number q of a stage into stage buffer `buf`: A's, then B's.  One LDS address (M0) serves four loads: three of them reach the next KiB by the immediate
  // offset, which moves the global address too: the bases sit 3 KiB low, the lane's offsets make up for what the immediate does not add.
  auto issue_codes = [&](auto qc, int buf) {
    constexpr int q = decltype(qc)::value, o = q < kMB ? q : q - kMB;
    load16_to_lds_at<(o & 3) * 1024>(voff[q], q < kMB ? base_a : base_b,
                                     lds0 + buf * kStageBytes + (q < kMB ? wave * (kMB * 1024) : kOperandBytes + wave * (kNB * 1024)) + (o & ~3) * 1024);
  };
  // The loads of a scale chunk (four K steps): 64 rows each, a wavefront's own of the first 256 (in a narrower tile some rows come twice, the same
  // bytes), and of a wider tile the last 64 by every wavefront (the count of its loads is one for all).
  auto issue_scales = [&]() {
    auto rows = [&](uint32_t first, int count, uint32_t last, const uint8_t* base, uint32_t dst) {
      const uint32_t r = static_cast<uint32_t>(min(static_cast<int>(first), count - 64));
      load16_to_lds(min(r + lane_srow, last + 7) * static_cast<uint32_t>(scale_ld), base, dst + r * 16);
    };
    rows(wave * 64, kTM, last_a, base_sa, scales0);
    rows(wave * 64, kTN, last_b, base_sb, scales0 + kTM * 16);
    if (kTN > 256) rows(256, kTN, last_b, base_sb, scales0 + kTM * 16);
  };

  const int stages = static_cast<int>(K / 256), chunks = static_cast<int>(K / 512);   // stages = 2 chunks >= 2
  int item = blockIdx.x;   // < num_tiles: the host launches at most that many workgroups
  int tm = 0, tn = 0;
  locate(item, tm, tn);
  aim(tm, tn, 0, 0);
  static_for<0, S::kLoads>([&](auto q) { issue_codes(q, 0); });
  base_a += kWideRowBytes;
  base_b += kWideRowBytes;
  static_for<0, S::kLoads>([&](auto q) { issue_codes(q, 1); });
  issue_scales();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  int4v fa[kMB], fb[kNB];
  // The scales of a chunk as read from LDS: lane l has the 16 bytes of row l & 15 of 16-row block 4 h + (l >> 4), h = 0 .. kA - 1 of A, then of B: a
  // read is 1 KiB of consecutive LDS.  Element e: the four scales of K step e.  (Some are of rows that count for nothing.)
  // Read as a dword per row and step, by all four lanes of a row, they took a third of the LDS's time: 8 instructions a step, two rows to a bank.
  int4v chunk[S::kA + S::kB];
  int scale[S::kA + S::kB];     // of the step that runs: byte t of number h: block 4 h + t of A; then of B
  float4v acc[kMB][kNB];
  bool stores_behind = false;   // the previous tile's stores were issued after the loads now in flight
  auto read_chunk = [&](auto qc) {
    constexpr int q = decltype(qc)::value;
    if constexpr (q < S::kA) lds_read_frag<q * 64 * 16, true>(chunk[q], a_scales);
    else lds_read_frag<(q - S::kA) * 64 * 16, true>(chunk[q], b_scales);
  };
  for (;;) {
    // The tile's first fragments and scales.  (After a tile of the same stream its last stage has read them already; they are
    // read again so that the output stage had their registers to work with.)
    static_for<0, S::kA + S::kB>(read_chunk);
    static_for<0, kR>([&](auto q) { lds_read_frag<decltype(q)::value * 16 * kWideRowBytes, true>(fa[decltype(q)::value], a_lo); });
    static_for<0, kNB>([&](auto q) { lds_read_frag<decltype(q)::value * 16 * kWideRowBytes, true>(fb[decltype(q)::value], b_lo); });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    static_for<0, S::kA + S::kB>([&](auto q) {
      arrived(chunk[decltype(q)::value]);
      scale[decltype(q)::value] = transpose_row(transpose_half(chunk[decltype(q)::value][0], sel_half), sel_row);
    });
    static_for<0, S::kA + S::kB>([&](auto q) { turned(scale[decltype(q)::value]); });
    asm volatile("s_nop 1");   // (see Schedule::turn)
    const int next_item = item + static_cast<int>(gridDim.x);
    const bool has_next = next_item < num_tiles;
    int next_tm = 0, next_tn = 0;
    if (has_next) locate(next_item, next_tm, next_tn);

    // One K step, number kS of its chunk (two stages of two steps).  The loads run two stages ahead of the MFMAs: a stage's buffer is free early in its second
    // step, and from there to the end of the step the loads of the stage after the next go into it; they have landed in the middle of the next stage's second step.  The scales of the
    // next chunk are loaded at the end of a chunk's first stage, into the place of its own, which are in registers.
    auto step = [&](auto first_tag, auto step_tag, int st) __attribute__((always_inline)) {
      constexpr bool kFirst = decltype(first_tag)::value;
      constexpr int kS = decltype(step_tag)::value, kBuf = kS >> 1;
      constexpr bool kSecond = kS & 1;
      constexpr uint32_t kCur = kBuf * kStageBytes, kNext = (kSecond ? kBuf ^ 1 : kBuf) * kStageBytes;
      const uint32_t a_cur = (kSecond ? a_hi : a_lo) + kCur, b_cur = (kSecond ? b_hi : b_lo) + kCur;
      const uint32_t a_nxt = (kSecond ? a_lo : a_hi) + kNext, b_nxt = (kSecond ? b_lo : b_hi) + kNext;
      static_for<0, kHalf>([&](auto nc) {
        constexpr int n = decltype(nc)::value, j = n / kR, i = (j & 1) ? kR - 1 - n % kR : n % kR, rd = S::upper_read(n);
        // Every third column: the B fragments of it and of the next two are back.  Behind them only the later ones, the last column's (read behind the
        // first MFMA) and A's have been issued.
        if constexpr (n % kR == 0 && j % 3 == 0 && !kFirst) {
          constexpr int last = j + 2 < kNB - 1 ? j + 2 : kNB - 1;
          constexpr int behind = n == 0 && S::lower_reads_behind_a() < kNB - 2 - last ? S::lower_reads_behind_a() : kNB - 2 - last + (n > 0);
          asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(last == kNB - 1 ? S::upper_reads_before(n) : behind + S::upper_reads_before(n)) : "memory");
        }
        if constexpr (kSecond && n == S::kFree) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
        }
        mfma_wide<kFirst, i * kNB + j < 64, (j & 3), (i & 3)>(acc[i][j], fb[j], fa[i], scale[S::kA + (j >> 2)], scale[i >> 2]);
        if constexpr (n == 0 && !kFirst) lds_read_frag<(kNB - 1) * 16 * kWideRowBytes, false>(fb[kNB - 1], b_cur);
        if constexpr (rd >= 0) lds_read_frag<(rd >= 0 ? rd : 0) * 16 * kWideRowBytes, kFirst>(fa[rd >= 0 ? rd : 0], a_cur);
        if constexpr (kSecond && n == 1) {
          // Where the loads go next: on within the tile, or to the next tile's first stage and chunk, or, with nothing
          // to follow, nowhere (the last stage and chunk are fetched again into buffers nobody reads any more).
          uint32_t advance = kWideRowBytes;
          if (kBuf == 0 && (st >> 1) + 1 < chunks) {
            base_sa += 16;
            base_sb += 16;
          }
          if (st + 2 == stages) {
            advance = 0;
            if (has_next) aim(next_tm, next_tn, 0, 0);
          } else if (st + 2 > stages && !has_next) {
            advance = 0;
          }
          base_a += advance;
          base_b += advance;
        }
        if constexpr (kSecond && n >= S::kFree) {
          constexpr int ld = S::load(n - S::kFree);
          if constexpr (ld >= 0) issue_codes(std::integral_constant<int, ld>{}, kBuf);
        }
      });
      // The lower half's A fragments are back; in a stage's second step the next stage has landed (its loads and scales: all but those of this step).
      if constexpr (kSecond) {
        if (kS == 1 && stores_behind && st == 0)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(S::kEarlyLoads + kTileStoresMx<kBf16Out, kNB> > 63 ? 63 : S::kEarlyLoads + kTileStoresMx<kBf16Out, kNB>) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(S::kEarlyLoads) : "memory");
        __builtin_amdgcn_s_barrier();
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
      uint32_t half[S::kA + S::kB];
      int next_scale[S::kA + S::kB];
      static_for<0, kHalf>([&](auto nc) {
        constexpr int n = decltype(nc)::value, j = n / kR, i = kR + ((j & 1) ? kR - 1 - n % kR : n % kR);
        constexpr int ra = S::lower_read_a(n), rb = S::lower_read_b(n), tr = S::turn(n);
        if constexpr (kS == 3 && n == S::kTurnFrom) {
          asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(S::lower_reads_before(n)) : "memory");
          static_for<0, S::kA + S::kB>([&](auto q) { arrived(chunk[decltype(q)::value]); });
        }
        mfma_wide<kFirst, i * kNB + j < 64, (j & 3), (i & 3)>(acc[i][j], fb[j], fa[i], scale[S::kA + (j >> 2)], scale[i >> 2]);
        if constexpr (kS == 3 && n < 2) static_for<n * 3, (n == 0 && S::kA + S::kB > 3 ? 3 : n * 3 > S::kA + S::kB ? n * 3 : S::kA + S::kB)>(read_chunk);
        if constexpr (ra >= 0) lds_read_frag<(ra >= 0 ? ra : 0) * 16 * kWideRowBytes, false>(fa[ra >= 0 ? ra : 0], a_nxt);
        if constexpr (rb >= 0) lds_read_frag<(rb >= 0 ? rb : 0) * 16 * kWideRowBytes, false>(fb[rb >= 0 ? rb : 0], b_nxt);
        if constexpr (tr >= 0 && tr % 2 == 0) {
          int v = chunk[tr / 2][(kS + 1) & 3];
          turned(v);   // (not ahead of this MFMA)
          half[tr / 2] = transpose_half(v, sel_half);
        }
        if constexpr (tr >= 0 && tr % 2 == 1) {
          next_scale[tr / 2] = transpose_row(half[tr / 2], sel_row);
          turned(next_scale[tr / 2]);
        }
        if constexpr (kSecond) {
          constexpr int ld = S::load(kHalf - S::kFree + n);
          if constexpr (ld >= 0) issue_codes(std::integral_constant<int, ld>{}, kBuf);
        }
      });
      if constexpr (kS == 1) issue_scales();
#pragma unroll
      for (int q = 0; q < S::kA + S::kB; ++q) scale[q] = next_scale[q];
    };
    auto chunk_of_steps = [&](auto first_tag, int st) __attribute__((always_inline)) {
      step(first_tag, std::integral_constant<int, 0>{}, st);
      step(std::false_type{}, std::integral_constant<int, 1>{}, st);
      step(std::false_type{}, std::integral_constant<int, 2>{}, st + 1);
      step(std::false_type{}, std::integral_constant<int, 3>{}, st + 1);
    };
    chunk_of_steps(std::true_type{}, 0);
    for (int st = 2; st < stages; st += 2) chunk_of_steps(std::false_type{}, st);

    // The MFMA results must have left the pipe before ordinary instructions read the accumulators (the compiler
    // cannot see into the assembly statements to insert these wait states itself), and the reads behind the last step must have arrived before
    // their registers serve anything else: the statements without an instruction keep the fragments until then and let the sums be used only from then on.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    static_for<0, kMB>([&](auto i) { keep(fa[decltype(i)::value]); });
    static_for<0, kNB>([&](auto j) { keep(fb[decltype(j)::value]); });
    static_for<0, kMB * kNB>([&](auto n) { settled<(decltype(n)::value < 64)>(acc[decltype(n)::value / kNB][decltype(n)::value % kNB]); });
    // With nothing to follow, the trailing global->LDS loads must have landed before the wavefront ends.
    if (!has_next) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // Everything below is computed here, per tile (see lane_setup).
    int wm = wave >> 1, wn = wave & 1;
    asm volatile("" : "+s"(wm), "+s"(wn));
    const int lane = lane_id();
    const TensorScales out_scale{A.ts, B.ts, false, false};    // both are 1 for MXFP4 (no tensor-level scale)
    const int64_t m0 = static_cast<int64_t>(tm) * kTM, n0 = static_cast<int64_t>(tn) * kTN;
    const int Mt = static_cast<int>(A.outer - m0 < kTM ? A.outer - m0 : kTM);
    const int Nt = static_cast<int>(B.outer - n0 < kTN ? B.outer - n0 : kTN);
    store_wave_block<kBf16Out, kNB>(acc, out_scale, Dv, ldd, accumulate, m0 + wm * (16 * kMB), n0 + wn * (16 * kNB), Mt - wm * (16 * kMB),
                                                     Nt - wn * (16 * kNB), lane);
    if (!has_next) break;
    stores_behind = Mt == kTM && Nt == kTN;   // every lane stored every block: the count is known
    item = next_item;
    tm = next_tm;
    tn = next_tn;
    lane_setup();
    aim(tm, tn, 1, 0);   // where the loads stand: the tile's second stage and first scale chunk are the last fetched
  }
}

}  // namespace

template <class Kernel>
static hipError_t launch_mx(Kernel kernel, PerDeviceOnce& once, int lds_bytes, const GemmArgs& g, dim3 grid, int tiles_m, int tiles_n,
                            hipStream_t s) {
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), lds_bytes, once);   // more dynamic LDS than the default limit
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds_bytes, s, g.a, g.b, g.K, g.d, g.ldd, g.accumulate, tiles_m, tiles_n);
  return hipGetLastError();
}

// Width of the k512 kernel's tiles: 256 rows x 32 nb columns.  A wider tile moves fewer bytes per product, but a product of a few
// hundred of them leaves CUs idle: a round of 256 tiles of nb = 10, 7, 5, 4 takes 1.19, 0.92, 0.75, 0.65 of one of nb = 8, and 0.9 of that where it does not fill the chip (fitted
// to 120 products), so the width with the smallest rounds x time is taken, the wider one of up to 256 columns at a tie.  Over these products it takes 0.4 % more than the best one.
// us per call at nb = 8 / 7 / 5 / 10: 4096 x 5120 x 5120 bf16 73.2 / 66.8 / 60.4 / 53.1, 5120 x 5120 x 4096 FP32 70.6 / 68.2 / 77.1 / 83.9, 2048 x 5120 x 5120 bf16 37.6 / 34.7 /
// 32.2 / 42.2, 8192 x 20480 x 5120 bf16 421 / 450 / 474 / 401.  (320 rows x 160 or 256 columns: no better over them.)
// 320 columns have to promise 2 %: five rounds of them in the place of six of 256, 0.8 % less by this estimate, took 1.02 times the time over 32 products (6656 x 14240 x 3584 bf16 186 us, 256
// columns 166; 9600 x 9216 x 6656 290 / 273); where they promise more, 0.94 over 368.
static int pick_mx_width(int64_t M, int64_t N) {
  constexpr int kWidths[5] = {8, 7, 5, 4, 10};
  constexpr double kTime[5] = {1.0, 0.92, 0.75, 0.65, 1.19};
  int best = 8;
  double best_time = 0.0;
  for (int i = 0; i < 5; ++i) {
    const int64_t tiles = ((M + TM - 1) / TM) * ((N + 32 * kWidths[i] - 1) / (32 * kWidths[i]));
    const double t = (tiles < 256 ? 0.9 : static_cast<double>((tiles + 255) / 256)) * kTime[i];
    if (i == 0 || t < (kWidths[i] == 10 ? 0.98 : 1.0) * best_time) {
      best = kWidths[i];
      best_time = t;
    }
  }
  return best;
}

template <int kNB>
static hipError_t launch_k512(const GemmArgs& g, int tiles_m, hipStream_t s) {
  static PerDeviceOnce once_bf16, once_f32;
  const int tiles_n = static_cast<int>((g.b.outer + 32 * kNB - 1) / (32 * kNB));
  const int64_t tiles = static_cast<int64_t>(tiles_m) * tiles_n;
  const dim3 grid(static_cast<unsigned>(tiles < 256 ? tiles : 256));   // one workgroup per CU, each running its tiles as one stream
  constexpr int lds = wide_lds_bytes(kNB);
  if (g.out_bf16) return launch_mx(gemm_mx_kernel_k512<true, kNB>, once_bf16, lds, g, grid, tiles_m, tiles_n, s);
  return launch_mx(gemm_mx_kernel_k512<false, kNB>, once_f32, lds, g, grid, tiles_m, tiles_n, s);
}

hipError_t launch_gemm_mx(const GemmArgs& g, hipStream_t s) {
  if (g.K >= (int64_t{1} << 24)) return hipErrorInvalidValue;   // the kernels' 32-bit byte offsets inside a block of rows
  const int tiles_m = static_cast<int>((g.a.outer + TM - 1) / TM), tiles_n = static_cast<int>((g.b.outer + TN - 1) / TN);
  // 16-byte pieces of scale rows need K / 32 to be a multiple of 16 and the scale arrays 16-byte aligned
  const bool wide = g.K % 512 == 0 && reinterpret_cast<uintptr_t>(g.a.scales) % 16 == 0 && reinterpret_cast<uintptr_t>(g.b.scales) % 16 == 0;
  if (wide) {
    switch (pick_mx_width(g.a.outer, g.b.outer)) {
      case 4: return launch_k512<4>(g, tiles_m, s);
      case 5: return launch_k512<5>(g, tiles_m, s);
      case 7: return launch_k512<7>(g, tiles_m, s);
      case 10: return launch_k512<10>(g, tiles_m, s);
      default: return launch_k512<8>(g, tiles_m, s);
    }
  }
  const dim3 grid(static_cast<unsigned>(tiles_m) * static_cast<unsigned>(tiles_n));
  static PerDeviceOnce set[2];
  if (g.out_bf16) return launch_mx(gemm_mx_kernel_any_k<true>, set[0], kLdsBytes, g, grid, tiles_m, tiles_n, s);
  return launch_mx(gemm_mx_kernel_any_k<false>, set[1], kLdsBytes, g, grid, tiles_m, tiles_n, s);
}

}  // namespace nvfp4

// For the tests, not part of the ABI: 32-column units of the tile that an MXFP4 product of these sizes takes where K is a multiple of 512.
extern "C" int nvfp4_internal_mx_gemm_width(int64_t M, int64_t N) { return nvfp4::pick_mx_width(M, N); }
