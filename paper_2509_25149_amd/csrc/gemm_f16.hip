// Two-pass form of the block-scaled GEMM (App. B.3 Eq. 5) for gfx950, used when
// the caller lends a workspace:
//   pass 1  decode both NVFP4 operands to FP16, value * block_scale (exact: the
//           product has at most 6 significant bits), into the workspace, in the
//           order pass 2 loads them;
//   pass 2  a plain FP16 x FP16 -> FP32 MFMA GEMM whose main loop has no VALU
//           work but address increments: tiles go from global memory straight
//           into LDS (global_load_lds_dwordx4), fragments come from LDS,
//           16x16x32 MFMAs (measured under the chip's power limit: a
//           register-only loop of v_mfma_f32_16x16x32_f16 sustains 12-20 % more
//           flop/s than one of v_mfma_f32_32x32x16_f16 on the same operand
//           values); a workgroup runs its tiles as one stream of K steps;
//   pass 3  only for a last, partial round of tiles, which pass 2 splits along
//           K: the sum of the partial tiles.
// Why: decoding inside the GEMM loop costs about one VALU instruction per
// element, and VALU instructions co-issued with MFMAs take matrix-pipe time
// (measured: the fused kernel runs at 1.0-1.07 PFLOP/s, this route at 1.5-1.6
// in the GEMM proper, the decode pass adding 5-8 % of its time).
// The results are identical to the fused kernel's up to FP32 summation order.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "nvfp4_internal.h"
#include "nvfp4_device.h"
#include "gemm_epilogue.h"

namespace nvfp4 {

namespace {

// ---------------------------------------------------------------- pass 1: decode
// Layout of a decoded operand ([outer, K] elements, outer a multiple of 16, K of 64): the piece the GEMM loads with
// one instruction and reads back as one MFMA fragment -- 16 rows x 32 k = 1 KiB -- is contiguous, the K steps of a
// 16-row block follow each other, and inside a piece the 16-byte chunks (8 k of one row) are in fragment order, the
// lane's order (lane l of an MFMA operand holds chunk l / 16 of row l % 16):
//   byte address of element (r, k) = ((r / 16) * (K / 32) + k / 32) * 1024 + (((k % 32) / 8) * 16 + r % 16) * 16 + (k % 8) * 2.
// So a load instruction reads 1 KiB of consecutive addresses into 1 KiB of consecutive LDS, and a fragment read is
// 1 KiB of consecutive LDS, lane l its bytes 16 l .. 16 l + 15: no bank conflicts, no swizzle.  (Measured with 8-row x
// 64-k pieces against rows of K * 2 bytes -- 8 separate 128-byte pieces per instruction, a stride that puts the
// pieces of all 256 tile rows into few cache channels: the GEMM's K step took 5-10 % less time on the three 12B
// shapes, same process, same data, identical results.)
//
// The decode pass: a workgroup takes a 16-row block x 512 k.  It reads the block's codes and scales row by row (256
// and 32 contiguous bytes per row), passes them through LDS, and writes 16 pieces of FP16 in output order, a thread
// 16 bytes at a time, consecutive threads consecutive addresses -- so that both sides of the pass move whole cache
// lines.  Both operands are decoded by one launch: the 16-row blocks of B follow those of A in the grid.
constexpr int kDecodeK = 512;                           // k per workgroup
constexpr int kDecodeCodeRow = kDecodeK / 2 + 16;       // bytes per row of codes in LDS; the 16 keep 16 rows off each other's banks
constexpr int kDecodeScaleRow = kDecodeK / 16 + 4;      // likewise for the scales
__global__ __launch_bounds__(256) void decode_f16_kernel(const uint8_t* __restrict__ a_codes,
                                                         const uint8_t* __restrict__ a_scales, int a_blocks,
                                                         _Float16* __restrict__ a_out,
                                                         const uint8_t* __restrict__ b_codes,
                                                         const uint8_t* __restrict__ b_scales, int b_blocks,
                                                         _Float16* __restrict__ b_out, int64_t K) {
  __shared__ __attribute__((aligned(16))) uint8_t lds_codes[16 * kDecodeCodeRow];
  __shared__ __attribute__((aligned(4))) uint8_t lds_scales[16 * kDecodeScaleRow];
  // consecutive workgroups walk along K: they read consecutive pieces of the same 16 rows and write consecutive 16 KiB
  const int k_groups = static_cast<int>((K + kDecodeK - 1) / kDecodeK);
  int blk = static_cast<int>(blockIdx.x) / k_groups;
  const int k_group = static_cast<int>(blockIdx.x) - blk * k_groups;
  const bool in_a = blk < a_blocks;
  if (!in_a) blk -= a_blocks;
  if (!in_a && blk >= b_blocks) return;
  const uint8_t* codes = in_a ? a_codes : b_codes;
  const uint8_t* scales = in_a ? a_scales : b_scales;
  half8v* out = reinterpret_cast<half8v*>(in_a ? a_out : b_out);
  const int t = static_cast<int>(threadIdx.x);
  const int64_t k0 = static_cast<int64_t>(k_group) * kDecodeK;
  {
    // codes: thread -> row t / 16, 32 elements (16 bytes) at k = k0 + 32 (t % 16)
    const int row = t >> 4, piece = t & 15;
    const int64_t k = k0 + piece * 32;
    if (k < K)
      *reinterpret_cast<uint4*>(lds_codes + row * kDecodeCodeRow + piece * 16) =
          *reinterpret_cast<const uint4*>(codes + ((static_cast<int64_t>(blk) * 16 + row) * K + k) / 2);
    // scales: threads 0..127 -> row t / 8, the four scale bytes of the 64 k from k0 + 64 (t % 8)
    if (t < 128) {
      const int srow = t >> 3, j = t & 7;
      if (k0 + j * 64 < K)
        *reinterpret_cast<uint32_t*>(lds_scales + srow * kDecodeScaleRow + j * 4) =
            *reinterpret_cast<const uint32_t*>(scales + ((static_cast<int64_t>(blk) * 16 + srow) * K + k0 + j * 64) / 16);
    }
  }
  __syncthreads();
  const int64_t pieces_per_block = K / 32;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    // 16-byte chunk number o of the workgroup's output: piece o / 64 (32 k each), chunk (o / 16) % 4 of it, row o % 16
    const int o = u * 256 + t;
    const int piece = o >> 6, chunk = (o >> 4) & 3, r16 = o & 15;
    if (k0 + piece * 32 >= K) break;
    const uint32_t c = *reinterpret_cast<const uint32_t*>(lds_codes + r16 * kDecodeCodeRow + piece * 16 + chunk * 4);
    const uint32_t s4 = *reinterpret_cast<const uint32_t*>(lds_scales + r16 * kDecodeScaleRow + (piece >> 1) * 4);
    const uint32_t scale = (s4 >> ((((piece & 1) * 2) + (chunk >> 1)) * 8)) & 0xffu;
    out[(static_cast<int64_t>(blk) * pieces_per_block + k0 / 32 + piece) * 64 + chunk * 16 + r16] = decode8_f16(c, e4m3_decode_f16x2(scale));
  }
}

// ---------------------------------------------------------------- pass 2: FP16 GEMM
// 32 kMB x 32 kNB outputs per workgroup, 256 threads = 4 wavefronts (2 x 2), one per SIMD, each 16 kMB x 16 kNB outputs as
// kMB x kNB MFMA 16x16 blocks: up to 400 accumulator registers, 256 of them in the accumulation half of the register file.
// LDS is a ring of four stages of 32 k, (A tile, B tile) as 2 kMB + 2 kNB pieces of 16 rows x 32 k.  A stage is
// filled by direct global->LDS loads: one instruction moves 64 lanes x 16 bytes, one piece of the decoded operand, into 1 KiB of consecutive LDS,
// which is one MFMA fragment in lane order.
//
// With one wavefront per SIMD nothing else can fill the matrix pipe while this one waits, so the loop is software-pipelined and its
// instruction order is fixed by hand (inline assembly keeps the compiler from regrouping it).  A stage runs the upper half of the
// wavefront's blocks column by column (down one, up the next: consecutive MFMAs share an operand; down every one took 1-2 % longer), then the lower half, and a fragment's registers take its next values as soon as its last MFMA has
// been issued: no second set of fragments, which is what leaves room for 160 x 160 outputs per wavefront.  Stage g, kMB / 2 * kNB MFMAs each:
//   upper half   behind them the reads of the lower half's A fragments of this stage, and the second half of the loads of stage g + 3
//   wait         own reads back (nobody needs this stage's buffer any more); own loads of stage g + 1 landed (those of g + 2 and g + 3 may
//                still be on their way); barrier
//   lower half   behind them the reads of the next stage's upper A fragments and of each B fragment as its column is done,
//                and the first half of the loads of stage g + 4, into the buffer of stage g
// so a load has two to three stages -- some 1.5 us -- to arrive in, and a fragment kMB / 2 * (kNB - 1) MFMAs, seven times what a read takes.
constexpr int TM = 256, TN = 256, TK = 64;       // TK: the unit K is split and counted in, two stages; TM, TN: the tiles of a split last round
constexpr int kThreads = 256;
constexpr int kStageK = 32;
constexpr int kPieceBytes = 16 * kStageK * 2;           // what one load instruction moves: 16 rows x 32 k, 1 KiB, contiguous in the decoded operand
constexpr int kStages = 4;
constexpr int stage_bytes(int mb, int nb) { return (2 * mb + (2 * nb + 3) / 4 * 4) * kPieceBytes; }   // (B's pieces rounded up to four wavefronts' loads)

template <int kBegin, int kEnd, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (kBegin < kEnd) {
    f(std::integral_constant<int, kBegin>{});
    static_for<kBegin + 1, kEnd>(f);
  }
}

// The MFMA's M index is the B row (n), its N index the A row (m): lane l ends up with the 4
// consecutive n = (l >> 4) * 4 .. + 3 of m = l & 15, which makes the output stores 64/128-bit.
// kAcc: the accumulator is pinned to the accumulation registers ("a"), which leaves the 256 ordinary registers to fragments, addresses and
// the accumulators beyond the 64th.  kFirst: the first of a work item, C = 0, so the accumulators are never cleared.
template <bool kFirst, bool kAcc>
__device__ __forceinline__ void mfma(float4v& acc, const half8v& b, const half8v& a) {
  if constexpr (kFirst && kAcc) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=a"(acc) : "v"(b), "v"(a));
  else if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=v"(acc) : "v"(b), "v"(a));
  else if constexpr (kAcc) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
  else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(b), "v"(a));
}

// No instruction: the value is used here / comes from here.
__device__ __forceinline__ void keep(const half8v& f) { asm volatile("" ::"v"(f)); }
template <bool kAcc>
__device__ __forceinline__ void settled(float4v& acc) {
  if constexpr (kAcc) asm volatile("" : "+a"(acc));
  else asm volatile("" : "+v"(acc));
}

// 16 bytes of LDS at addr + kOff.  Asynchronous: the caller waits (lgkmcnt) before the value is used.  kNew: into any registers; else
// into those that the fragment has (an operand in and out).
template <int kOff, bool kNew = false>
__device__ __forceinline__ void lds_read16(half8v& dst, uint32_t addr) {
  if constexpr (kNew) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(dst) : "v"(addr), "n"(kOff));
  else asm volatile("ds_read_b128 %0, %1 offset:%2" : "+v"(dst) : "v"(addr), "n"(kOff));
}

// 64 lanes x 16 bytes from global memory (wave-uniform base + per-lane 32-bit offset) straight into 1 KiB of consecutive LDS
// starting at the wave-uniform LDS address lds_dst + kOff.  Asynchronous (vmcnt).  kOff is the instruction's immediate offset, which is added to the LDS
// address and to the global address alike, so the caller passes a base that is kOff too low.  M0, the LDS address, is an operand: where a
// following load has the same lds_dst the compiler sets it once for both, and whatever else it may put into M0 in between it undoes.  (s_nop: the wait
// state that M0 needs when it has just been set.)
template <int kOff>
__device__ __forceinline__ void load_1k_to_lds(uint32_t lane_offset, const char* base_minus_off, uint32_t lds_dst) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(lane_offset), "s"(base_minus_off), "n"(kOff), "{m0}"(lds_dst) : "memory");
}

// A wavefront's output stage issues kMB ceil(kNB / 2) (bf16) or kMB kNB (FP32) stores for a full tile (store_wave_block: 16 bytes
// per lane and instruction).  Three quarters of them: the number of its memory operations that may still be
// outstanding when the loads issued before it are needed, with a margin against a store more or less.
template <bool kBf16Out, int kMB, int kNB>
constexpr int kTileStores = (kMB * 3 / 4) * (kBf16Out ? (kNB + 1) / 2 : kNB);

// What goes behind the MFMAs of a stage.  kR = kMB / 2 rows of blocks a half; MFMA n of a half is column n / kR, row n % kR.
template <int kMB, int kNB>
struct Schedule {
  static constexpr int kR = kMB / 2, kHalf = kR * kNB;
  static constexpr int kALoads = kMB / 2, kBLoads = (2 * kNB + 3) / 4, kLoads = kALoads + kBLoads;   // a wavefront's loads per stage (some of the last wavefront's of B are not needed)
  static constexpr int kEarly = (kLoads + 1) / 2;   // of them in the lower half, the rest in the upper half of the following stage
  // upper half: which A fragment of the lower half is read behind MFMA n, or -1; the last of them is back when the half ends
  static constexpr int kGap = kHalf - 16 >= 2 * kR ? (kHalf - 16) / kR : 1;
  static constexpr int upper_read(int n) { return n >= 1 && (n - 1) % kGap == 0 && (n - 1) / kGap < kR ? kR + (n - 1) / kGap : -1; }
  // lower half: which upper A fragment of the next stage (all of them before the last two of B), and which B fragment
  static constexpr int kGapA = 2 + kR * (kR - 1) < kR * (kNB - 2) ? kR : 3;
  static_assert(2 + kGapA * (kR - 1) < kR * (kNB - 2), "the last two reads of a stage are of B");
  static constexpr int lower_read_a(int n) { return n >= 2 && (n - 2) % kGapA == 0 && (n - 2) / kGapA < kR ? (n - 2) / kGapA : -1; }
  static constexpr int lower_read_b(int n) { return n >= kR && n % kR == 0 ? n / kR - 1 : -1; }   // (the last column's: behind the next stage's first MFMA)
  static constexpr int lower_reads_behind_a() {   // of B
    int r = 0;
    for (int k = 2 + kGapA * (kR - 1); k < kHalf; ++k) r += lower_read_b(k) >= 0;
    return r;
  }
  // how many of the upper half's reads of A are behind the MFMAs before n
  static constexpr int upper_reads_before(int n) {
    int r = 0;
    for (int k = 0; k < n; ++k) r += upper_read(k) >= 0;
    return r;
  }
  static_assert(upper_reads_before(kHalf) == kR, "");
  // which of `count` loads goes behind MFMA n: evenly spread, half a distance in
  static constexpr int load(int n, int count) {
    const int at = n * count + kHalf / 2;
    return (at + count) / kHalf > at / kHalf ? at / kHalf : -1;
  }
};

// Tiles [tile_begin, tile_begin + tile_count) of the tiling are covered.
//
// k_splits == 1: a workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ... of the launch (the host launches one
// workgroup per CU when there are more tiles than CUs) and runs them as ONE stream of stages: the loads issued during a
// tile's last four stages already fetch the next tile's first four, so that the pipeline neither drains nor refills at
// a tile boundary -- what remains there is reading the sums out, scaling, converting and issuing the stores,
// which then drain under the next tile's MFMAs (measured with timestamps in the one-tile-per-workgroup form: 4.2 us
// of pipeline fill, 5.5 us of output stage, most of it waiting for the stores of all CUs at once, and 0.6 us between
// workgroups, per 118 us of main loop at K = 5120).  Needs K >= 4 stages (2 K steps of 64); the host launches one workgroup per tile
// otherwise.
//
// k_splits > 1 (one work item per workgroup) fills the chip during a last, partial round of tiles: a tile is shared by
// k_splits workgroups, each summing one contiguous range of K steps and storing its FP32 partial tile to
// `partials`; splitk_sum_kernel, launched behind this one, adds the partials in split order and stores the tiles.
// (The sum used to be done here, by whichever workgroup of a tile finished last, found by a ticket counter: by
// timestamps inside the kernel, of the 127 us such a launch took on 64 tiles x 4 splits at K = 8192, the K steps
// were 48, the partial stores 7, the device-wide fence and the ticket 10, and one workgroup fetching and adding the
// 1 MiB that four XCDs had written 50 -- with 16 loads in flight per thread, and 90 with 64.)
// kRowScales: an operand carries a tensor-level scale per row (uniform over a launch, and a different output stage).
// kSplit: k_splits > 1; the output stage is the store of the partial tile (kBf16Out and kRowScales are false then).
// kMB, kNB: 16-row and 16-column blocks per wavefront; which tile a product takes: pick_tile.
template <bool kBf16Out, bool kRowScales, bool kSplit, int kMB, int kNB>
__global__ __launch_bounds__(kThreads) void gemm_f16_kernel(const _Float16* __restrict__ A, const _Float16* __restrict__ B,
                                                            int64_t M, int64_t N, int64_t K, const float* __restrict__ a_ts,
                                                            const float* __restrict__ b_ts, void* __restrict__ Dv,
                                                            int64_t ldd, bool accumulate, int tiles_m, int tiles_n,
                                                            int tile_begin, int tile_count, int k_splits, float* partials,
                                                            bool a_ts_per_row, bool b_ts_per_row) {
  using S = Schedule<kMB, kNB>;
  constexpr int kTM = 32 * kMB, kTN = 32 * kNB, kStageBytes = stage_bytes(kMB, kNB);
  constexpr int kR = S::kR, kHalf = S::kHalf, kALoads = S::kALoads, kBLoads = S::kBLoads, kLoads = S::kLoads, kEarly = S::kEarly;
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);

  // Work item -> tile: consecutive workgroup ids go to different XCDs (round robin over 8, one L2 each);
  // give every XCD a contiguous range of tiles, walked in bands of 8 tile rows.  (With one workgroup per CU the ids
  // of a later round continue the first round's, 8 | gridDim.x, so the low three bits stay the XCD.)
  auto locate = [&](int wg, int& tm, int& tn) -> int {
    if ((tile_count & 7) == 0) wg = (wg & 7) * (tile_count >> 3) + (wg >> 3);
    tile_coordinates(tile_begin + wg, tiles_m, tiles_n, tm, tn);
    return wg;   // the tile's number within the launch
  };

  // Direct-load sources: load q of wavefront w fills 16 rows of a tile (block w * kALoads + q of A's, w * kBLoads + q of B's), which the decoded
  // operand holds as 1 KiB of consecutive bytes per stage, in LDS order (lane l: bytes 16 l .. 16 l + 15).  An address
  // is a wave-uniform 64-bit base per operand, which holds the tile and the stage being fetched, plus a per-lane
  // 32-bit offset per instruction (320 rows of K * 2 bytes: K < 2^21, checked on the host), which holds the 16-row
  // block and does not change within a tile: moving on by a stage is two scalar additions per operand.  (Every
  // vector instruction between two MFMAs costs: with the stage added to the 8 per-lane offsets instead, the three
  // 12B GEMM calls took 2 % longer.)  A block past the end of an operand is replaced by the operand's last block
  // (rows come in multiples of 16); it only feeds outputs that are never stored.
  // One instruction per load inside the loop (a single wavefront per SIMD issues in order: what it spends on anything
  // else, the matrix pipe waits): M0, the LDS destination, is written once per four loads of an operand; the others reach
  // the next KiB through the instruction's immediate offset, which moves the LDS and the global address alike, so
  // the bases sit 3 KiB low and the offsets make up for what the immediate does not add.
  //
  // What depends on the lane is worked out once per tile, from a lane number asked for on the spot: values the
  // compiler could keep from before the first tile would have to live through every output stage, which needs the
  // registers itself, and end up in scratch memory, to be fetched back inside the K steps.
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  uint32_t lane_bytes = 0;          // the lane's part of a load offset
  uint32_t a_frag = 0, b_frag = 0;  // the lane's 16 bytes of the wavefront's first A / B fragment in the buffer that is read from
  auto lane_setup = [&](uint32_t buf) {
    lane_bytes = static_cast<uint32_t>(lane_id()) * 16u;
    a_frag = lds0 + buf * kStageBytes + (wave >> 1) * (kMB * kPieceBytes) + lane_bytes;
    b_frag = lds0 + buf * kStageBytes + 2 * kMB * kPieceBytes + (wave & 1) * (kNB * kPieceBytes) + lane_bytes;
  };
  lane_setup(0);
  const char* base_a = nullptr;
  const char* base_b = nullptr;
  uint32_t voff[kLoads];   // A's, then B's
  // Point the loads at stage st (32 k) of tile (tm, tn).
  auto aim = [&](int tm, int tn, int st) {
    const int64_t m_first = static_cast<int64_t>(tm) * kTM, n_first = static_cast<int64_t>(tn) * kTN;
    base_a = reinterpret_cast<const char*>(A) + m_first * K * 2 + (st - 3) * kPieceBytes;
    base_b = reinterpret_cast<const char*>(B) + n_first * K * 2 + (st - 3) * kPieceBytes;
    // 16-row blocks counted from the tile's first; a block's stages are K / 32 KiB
    const uint32_t last_a = static_cast<uint32_t>(M - 16 - m_first) >> 4, last_b = static_cast<uint32_t>(N - 16 - n_first) >> 4;
#pragma unroll
    for (int q = 0; q < kALoads; ++q)
      voff[q] = lane_bytes + min(static_cast<uint32_t>(wave * kALoads + q), last_a) * static_cast<uint32_t>(K * 32) + static_cast<uint32_t>(3 - (q & 3)) * 1024u;
#pragma unroll
    for (int q = 0; q < kBLoads; ++q)
      voff[kALoads + q] = lane_bytes + min(static_cast<uint32_t>(wave * kBLoads + q), last_b) * static_cast<uint32_t>(K * 32) + static_cast<uint32_t>(3 - (q & 3)) * 1024u;
  };
  const uint32_t fill_a = lds0 + wave * (kALoads * kPieceBytes), fill_b = lds0 + (2 * kMB + wave * kBLoads) * kPieceBytes;   // this wavefront's pieces of each operand tile
  // load q of the wavefront's that fill ring buffer `buf`
  auto issue = [&](auto qc, uint32_t buf) {
    constexpr int q = decltype(qc)::value, o = q < kALoads ? q : q - kALoads;
    load_1k_to_lds<(o & 3) * 1024>(voff[q], q < kALoads ? base_a : base_b, (q < kALoads ? fill_a : fill_b) + (o & ~3) * kPieceBytes + buf * kStageBytes);
  };

  const int KT = static_cast<int>(K / TK);
  const int items = tile_count * k_splits;
  int item = blockIdx.x;   // < items: the host launches at most that many workgroups
  int tm = 0, tn = 0;
  const int split = item % k_splits;   // k_splits > 1: one work item per workgroup
  const int tile_local = locate(item / k_splits, tm, tn);
  const int kt_begin = static_cast<int>(static_cast<int64_t>(KT) * split / k_splits);
  const int kt_end = static_cast<int>(static_cast<int64_t>(KT) * (split + 1) / k_splits);   // > kt_begin: KT >= k_splits
  const int stages = 2 * (kt_end - kt_begin), st_end = 2 * kt_end;   // of an item (with k_splits == 1 the same for every tile)
  // The stage the loads were last pointed at: they run up to four stages ahead of the MFMAs.
  int fetch_st = 2 * kt_begin;
  aim(tm, tn, fetch_st);
  static_for<0, kLoads>([&](auto q) { issue(q, 0); });
#pragma unroll
  for (uint32_t buf = 1; buf < kStages; ++buf) {
    if (fetch_st + 1 < st_end) {   // (an item of two stages fetches its last three times)
      ++fetch_st;
      base_a += kPieceBytes;
      base_b += kPieceBytes;
    }
    // (the last stage's second half: behind the first MFMAs, as in every later stage)
    static_for<0, kLoads>([&](auto q) {
      if (buf + 1 < kStages || decltype(q)::value < kEarly) issue(q, buf);
    });
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoads + kEarly) : "memory");   // the first stage
  __builtin_amdgcn_s_barrier();

  half8v fa[kMB], fb[kNB];
  float4v acc[kMB][kNB];
  uint32_t g = 0;               // stages done so far; stage g lives in ring buffer g % 4
  bool stores_behind = false;   // the previous tile's kTileStores stores were issued after the loads now in flight
  for (;;) {
    // The tile's first fragments.  (After a tile of the same stream its last stage has read them already; they are read
    // again so that the output stage had their registers to work with.)
    static_for<0, kR>([&](auto q) { lds_read16<decltype(q)::value * kPieceBytes, true>(fa[decltype(q)::value], a_frag); });
    static_for<0, kNB>([&](auto q) { lds_read16<decltype(q)::value * kPieceBytes, true>(fb[decltype(q)::value], b_frag); });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // The next tile of this workgroup, if any: its stages follow this tile's without a break (k_splits == 1 then).
    const int next_item = item + static_cast<int>(gridDim.x);
    const bool has_next = next_item < items;
    int next_tm = 0, next_tn = 0;
    if (has_next) locate(next_item, next_tm, next_tn);

    // One stage.  kFirst: the item's first (accumulators
    // start from zero); kRelaxed: one of its first two (the stores of the tile before may still be in flight behind
    // the loads this stage waits for).
    auto stage = [&](auto first_tag, auto relaxed_tag) {
      constexpr bool kFirst = decltype(first_tag)::value, kRelaxed = decltype(relaxed_tag)::value;
      const uint32_t buf = g & 3u, before = (g - 1u) & 3u;
      static_for<0, kHalf>([&](auto nc) {
        constexpr int n = decltype(nc)::value, j = n / kR, i = (j & 1) ? kR - 1 - n % kR : n % kR, rd = S::upper_read(n), ld = S::load(n, kLoads - kEarly);
        // Every third column: the B fragments of it and of the next two are back.  Behind them only the later ones, the last column's (read behind the
        // first MFMA) and A's have been issued.
        if constexpr (n % kR == 0 && j % 3 == 0 && !kFirst) {
          constexpr int last = j + 2 < kNB - 1 ? j + 2 : kNB - 1;
          constexpr int behind = n == 0 && S::lower_reads_behind_a() < kNB - 2 - last ? S::lower_reads_behind_a() : kNB - 2 - last + (n > 0);
          asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(last == kNB - 1 ? S::upper_reads_before(n) : behind + S::upper_reads_before(n)) : "memory");
        }
        mfma<kFirst, i * kNB + j < 64>(acc[i][j], fb[j], fa[i]);
        if constexpr (n == 0 && !kFirst) lds_read16<(kNB - 1) * kPieceBytes>(fb[kNB - 1], b_frag);
        if constexpr (rd >= 0) lds_read16<(rd >= 0 ? rd : 0) * kPieceBytes, kFirst>(fa[rd >= 0 ? rd : 0], a_frag);
        if constexpr (ld >= 0) issue(std::integral_constant<int, kEarly + (ld >= 0 ? ld : 0)>{}, before);
      });
      // Memory operations complete in issue order.  Behind the loads of stage g + 1 this wavefront has issued those of
      // g + 2 and g + 3, kLoads each, and, across a tile boundary, the stores of the tile before.
      // (The reads are waited for on every path, whatever is known of the stores.)
      constexpr int kBehind = 2 * kLoads + (kRelaxed ? kTileStores<kBf16Out, kMB, kNB> : 0);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kBehind > 63 ? 63 : kBehind) : "memory");
      if (kRelaxed && !stores_behind) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoads) : "memory");
      __builtin_amdgcn_s_barrier();
      // The loads move on one stage: within the tile, or to the next tile's stage 0, or, with nothing to follow, not at
      // all (the last stage is fetched again, into a buffer nobody reads any more: no branches around the loads).
      uint32_t advance = kPieceBytes;
      if (fetch_st + 1 < st_end) {
        ++fetch_st;
      } else {
        advance = 0;
        if (has_next) {
          fetch_st = 0;
          aim(next_tm, next_tn, 0);
        }
      }
      const uint32_t to_next = buf == kStages - 1 ? static_cast<uint32_t>(-(kStages - 1) * kStageBytes) : static_cast<uint32_t>(kStageBytes);
      static_for<0, kHalf>([&](auto nc) {
        constexpr int n = decltype(nc)::value, j = n / kR, i = kR + ((j & 1) ? kR - 1 - n % kR : n % kR), ra = S::lower_read_a(n), rb = S::lower_read_b(n), ld = S::load(n, kEarly);
        mfma<kFirst, i * kNB + j < 64>(acc[i][j], fb[j], fa[i]);
        if constexpr (n == 0) {
          a_frag += to_next;
          b_frag += to_next;
          base_a += advance;
          base_b += advance;
        }
        if constexpr (ra >= 0) lds_read16<(ra >= 0 ? ra : 0) * kPieceBytes>(fa[ra >= 0 ? ra : 0], a_frag);
        if constexpr (rb >= 0) lds_read16<(rb >= 0 ? rb : 0) * kPieceBytes>(fb[rb >= 0 ? rb : 0], b_frag);
        if constexpr (ld >= 0) issue(std::integral_constant<int, ld>{}, buf);
      });
      ++g;
    };
    stage(std::true_type{}, std::true_type{});
    stage(std::false_type{}, std::true_type{});
    for (int st = 2; st < stages; ++st) stage(std::false_type{}, std::false_type{});

    // The MFMA results must have left the pipe before ordinary instructions read the accumulators (the compiler
    // cannot see into the assembly statements to insert these wait states itself), and the reads behind the last stage must have arrived before
    // their registers serve anything else: the statements without an instruction keep the fragments until then and let the sums be used only from then on.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    static_for<0, kMB>([&](auto i) { keep(fa[decltype(i)::value]); });
    static_for<0, kNB>([&](auto j) { keep(fb[decltype(j)::value]); });
    static_for<0, kMB * kNB>([&](auto n) { settled<(decltype(n)::value < 64)>(acc[decltype(n)::value / kNB][decltype(n)::value % kNB]); });
    // With nothing to follow, the trailing global->LDS loads must have landed before the wavefront ends; otherwise the next
    // tile's first stage is in LDS by now and three more on their way there.
    if (!has_next) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }

    // Everything below is computed here, per tile: were the compiler to move the output stage's loop-invariant
    // address arithmetic in front of the stream, it would have to keep it in registers through the K steps, which
    // have none to spare.
    int wm = wave >> 1, wn = wave & 1;
    asm volatile("" : "+s"(wm), "+s"(wn));
    const int lane = lane_id(), tid = (wm * 2 + wn) * 64 + lane;
    // Tensor-level decode scales on the finished sums (App. B.3, after Eq. 5).
    const TensorScales out_scale{a_ts, b_ts, a_ts_per_row, b_ts_per_row};
    const int64_t m0 = static_cast<int64_t>(tm) * kTM, n0 = static_cast<int64_t>(tn) * kTN;
    const int Mt = static_cast<int>(M - m0 < kTM ? M - m0 : kTM);
    const int Nt = static_cast<int>(N - n0 < kTN ? N - n0 : kTN);

    if constexpr (kSplit) {   // has_next is false
      static_assert(kMB == 8 && kNB == 8, "the partial tiles are 256 x 256");
      // Partial tile in fragment order: float4 number (i * 8 + j) * 256 + tid.
      float4v* mine = reinterpret_cast<float4v*>(partials) +
                      (static_cast<int64_t>(tile_local) * k_splits + split) * (TM * TN / 4) + tid;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < kNB; ++j) mine[(i * kNB + j) * kThreads] = acc[i][j];
      return;
    } else {
      store_wave_block_impl<kBf16Out, kRowScales, kMB, kNB>(acc, out_scale, Dv, ldd, accumulate, m0 + wm * (16 * kMB), n0 + wn * (16 * kNB),
                                                            Mt - wm * (16 * kMB), Nt - wn * (16 * kNB), lane);
    }
    if (!has_next) break;
    stores_behind = Mt == kTM && Nt == kTN;   // every lane stored every block: the count is known
    item = next_item;
    tm = next_tm;
    tn = next_tn;
    lane_setup(g & 3u);
    aim(tm, tn, fetch_st);
  }
}

// The sums over K of the tiles a split-K launch covered: one wavefront per tile, 128 x 128 block of it (the block one
// wavefront of gemm_f16_kernel holds, in the same register layout, which is the order the partial tiles are stored
// in) and 16 rows of that, sum = ((p0 + p1) + p2) + ... in split order, then the same output stage.  Many small
// workgroups: the partial tiles were written by other XCDs and every load of them is a long trip, so what counts is
// how many are in flight over the chip (with a wavefront per 128 x 128 block the sum of 64 tiles x 4 splits took 57 us).
template <bool kBf16Out, bool kRowScales>
__global__ __launch_bounds__(64) void splitk_sum_kernel(const float* __restrict__ partials, int k_splits, int64_t M, int64_t N,
                                                        const float* __restrict__ a_ts, const float* __restrict__ b_ts,
                                                        void* __restrict__ Dv, int64_t ldd, bool accumulate, int tiles_m,
                                                        int tiles_n, int tile_begin, bool a_ts_per_row, bool b_ts_per_row) {
  const int tile_local = static_cast<int>(blockIdx.x) >> 5, wave = (static_cast<int>(blockIdx.x) >> 3) & 3;
  const int i = static_cast<int>(blockIdx.x) & 7;
  const int lane = static_cast<int>(threadIdx.x), wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_coordinates(tile_begin + tile_local, tiles_m, tiles_n, tm, tn);
  // float4 number (i * 8 + j) * 256 + 64 wave + lane of a partial tile
  const float4v* all = reinterpret_cast<const float4v*>(partials) +
                       static_cast<int64_t>(tile_local) * k_splits * (TM * TN / 4) + i * 8 * kThreads + wave * 64 + lane;
  float4v sums[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) sums[j] = all[j * kThreads];
  for (int sp = 1; sp < k_splits; ++sp) {
    const float4v* part = all + static_cast<int64_t>(sp) * (TM * TN / 4);
    float4v t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = part[j * kThreads];
#pragma unroll
    for (int j = 0; j < 8; ++j) sums[j] = sums[j] + t[j];
  }
  const TensorScales ts{a_ts, b_ts, a_ts_per_row, b_ts_per_row};
  const int64_t m0 = static_cast<int64_t>(tm) * TM, n0 = static_cast<int64_t>(tn) * TN;
  const int Mt = static_cast<int>(M - m0 < TM ? M - m0 : TM);
  const int Nt = static_cast<int>(N - n0 < TN ? N - n0 : TN);
  const WaveBlockStore<kBf16Out, kRowScales> out(ts, Dv, ldd, accumulate, m0 + wm * 128, n0 + wn * 128, Mt - wm * 128,
                                                 Nt - wn * 128, lane);
  out.store_rows(sums, i, kRowScales ? out.row_scale(ts, m0 + wm * 128, i) : 0.0f);
}

}  // namespace

// Workspace: [A as FP16][B as FP16][split-K partial tiles], each part 256-byte aligned.
constexpr int kCUs = 256;
constexpr size_t kPartialTileBytes = static_cast<size_t>(TM) * TN * sizeof(float);

// How the last, partial round of 256x256 tiles is run where a product takes those: `tail` tiles (0 = there is none to treat
// specially) shared by `splits` workgroups each.
struct TailPlan {
  int tail, splits;
};

static TailPlan plan_tail(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ((M + TM - 1) / TM) * ((N + TN - 1) / TN);
  TailPlan p{static_cast<int>(tiles % kCUs), 1};
  if (tiles < kCUs || p.tail == 0) return TailPlan{0, 1};
  const int64_t KT = K / TK;
  while (p.splits < 8 && p.tail * (p.splits * 2) <= kCUs && KT / (p.splits * 2) >= 8) p.splits *= 2;
  if (p.splits == 1) p.tail = 0;
  return p;
}

// Tile width (32 nb columns) of the whole product in tiles of 256 rows and at most 256 columns, and how long it takes in rounds of 256 x 256 tiles.  A narrower tile takes
// 0.90, 0.80, 0.68 of the time for nb = 7, 6, 5 (fewer products per byte moved), but rounds come out better for some
// products; the widest wins a tie.  A split last round costs its share of a round and 0.15 for the partial tiles.  Measured,
// us per call with nb = 8 / 7 / 6 / 5: 5120 x 5120 x 4096 (FP32) 192 / 179 / 216 / 193, 2048 x 5120 x 5120 113 / 104 / 95 / 93, 4096 x 5120 x 5120
// 171 (split) / 189 / 170 / 160, 3072 x 5120 x 5120 118 / 187 / 166 / 147, 8192 x 5120 x 20480 1165 (split) / 1225 / 1337 / 1337.
struct Width {
  int nb;
  double rounds;
  int64_t tiles;
};
// A product that is accumulated into its result takes longer over the result the more tiles there are (5120 x 20480, K = 64 / 256 / 512: nb = 8
// 283 / 299 / 333, nb = 5 306 / 313 / 345): there a narrower tile has to promise 4 % while K is short (`reluctant`; no last round is split
// then, so the sums are the same), and a larger one more (promise_needed; 320 x 320 there 287 / 293 / 315).
static Width pick_width(int64_t M, int64_t N, const TailPlan& p, bool reluctant) {
  constexpr double kTime[4] = {1.0, 0.90, 0.80, 0.68};
  const int64_t tiles_m = (M + TM - 1) / TM;
  Width best{8, 0.0, 0};
  for (int i = 0; i < 4; ++i) {
    const int nb = 8 - i;
    const int64_t tiles = tiles_m * ((N + 32 * nb - 1) / (32 * nb));
    double rounds = static_cast<double>((tiles + kCUs - 1) / kCUs);
    if (i == 0 && p.tail) rounds = static_cast<double>((tiles - p.tail) / kCUs) + 1.0 / p.splits + 0.15;
    rounds *= kTime[i];
    if (i == 0 || rounds < (reluctant && best.nb == 8 ? 0.96 : 1.0) * best.rounds) best = Width{nb, rounds, tiles};
  }
  return best;
}

// What a product takes in tiles of 32 mb x 32 nb, us, without the decode pass: rounds of 256 tiles at `result` us and `k` of the 256 x 256 tile's time per k, which is
// 14.9 ns while there are fewer tiles than CUs and 17.0 when the chip is full (the clock drops with the matrix pipes busy).  Fitted to 780 times (130 products of
// 12 us to 1.3 ms, six tiles each), which it meets within 6.5 % (standard deviation).
struct TileTime {
  int mb, nb;
  double result, k;
};
constexpr TileTime kTileTimes[] = {{8, 8, 7.8, 1.0}, {8, 7, 7.1, 0.912}, {8, 6, 6.3, 0.80}, {8, 5, 5.4, 0.692}, {8, 10, 8.6, 1.242}, {10, 10, 9.9, 1.51}};
static double tile_us(const TileTime& t, int64_t tiles, double rounds, int64_t K) {
  return rounds * (t.result + static_cast<double>(K) * t.k * (tiles >= kCUs ? 0.0170 : 0.0149));
}
static double rounds_of(int64_t tiles) { return static_cast<double>((tiles + kCUs - 1) / kCUs); }

// The tile of a product, starting from its width among the tiles of 256 rows: 256 x 320 and 320 x 320 where they take less.  A byte that is loaded or read from LDS serves
// 1.11 and 1.25 times the MFMAs of a 256 x 256 tile, and for many products rounds come out better.  us per call, the best of the others / 256 x 320 / 320 x 320:
// 8192 x 20480 x 5120 bf16 1131 / 1112 / 1137, 8192 x 5120 x 20480 1200 / 1152 / 1251, 5120 x 20480 x 8192 FP32 1243 / 1201 / 1127, 5120 x 5120 x 4096 FP32 188 / 217 / 154,
// 4096 x 15360 x 2048 bf16 192 / 178 / 207.  Over the 130 products the tile with the smallest estimate takes 0.1 % more than the best one.
// A larger tile has no round split, and tiles without a split sum in the same order.
// (320 x 320 with a scale per row: the output stage has too few registers for the scales.)
// Where the contraction is short the result is most of the work, which the estimate knows least about: there a larger tile has to promise more, most of all where the
// result is accumulated (read too).  Measured, time in the tile of 256 rows over that in the larger one, geometric mean and least, by what the estimate promises: accumulated,
// K < 1024, 256 x 320 under 0.9 1.06, 0.98, from 0.9 on 0.98, 0.88; 320 x 320 under 0.8 1.04, 0.95, from 0.8 on 0.96, 0.84; plain results, K < 400, from 0.95 on
// 0.95, 0.92 (FP32), 0.98, 0.94 (bf16).  13312 x 1296 x 512 accumulated: 256 x 160 48 us, 320 x 320 56.  And 320 x 320 in the place of 256 x 160, one round of about 215 for two
// of nearly 256 each, has to promise a tenth: 8448 x 2288 x 1216 accumulated 66 / 74, 6432 x 3008 x 1024 FP32 41.5 / 43.5 with promises of 0.95, 20336 x 2320 x 1024 1.12 times
// faster with one of 0.83.
static double promise_needed(int mb, int units, int64_t K, bool accumulate) {
  if (accumulate && K < 1024) return mb == 8 ? 0.9 : 0.8;
  if (mb == 10 && units == 5) return 0.9;
  return K < 400 ? 0.95 : 1.0;
}
struct Tile {
  int mb, nb;
  double gain;   // time in it over that in the tile of 256 rows
};
static Tile pick_tile(int64_t M, int64_t N, int64_t K, const Width& w, const TailPlan& tail, bool row_scales, bool accumulate) {
  Tile best{8, w.nb, 1.0};
  double base = 0.0;   // (the tile of 256 rows comes first)
  for (const TileTime& t : kTileTimes) {
    const int64_t tiles = ((M + 32 * t.mb - 1) / (32 * t.mb)) * ((N + 32 * t.nb - 1) / (32 * t.nb));
    double rounds = rounds_of(tiles);
    if (t.nb <= 8) {
      if (t.nb != w.nb) continue;
      if (w.nb == 8 && tail.tail) rounds = static_cast<double>((tiles - tail.tail) / kCUs) + 1.0 / tail.splits + 0.3;   // (the partial tiles)
    } else if (row_scales && t.mb == 10) {
      continue;
    }
    const double us = tile_us(t, tiles, rounds, K);
    if (t.nb <= 8) base = us;
    else if (us < best.gain * base && us < promise_needed(t.mb, w.nb, K, accumulate) * base) best = Tile{t.mb, t.nb, us / base};
  }
  return best;
}

// FP16 bytes of the operands that still have to be decoded into the workspace (rows_a / rows_b: 0 for an operand the
// caller has decoded beforehand)
static size_t operand_bytes(int64_t rows_a, int64_t rows_b, int64_t K) {
  const size_t b = static_cast<size_t>(rows_a + rows_b) * static_cast<size_t>(K) * 2;
  return (b + 255) & ~static_cast<size_t>(255);
}

static size_t partial_bytes(const TailPlan& p) { return static_cast<size_t>(p.tail) * p.splits * kPartialTileBytes; }

// The tile of a product and what goes with it: how many tiles of its last round are split (of 256 x 256 tiles only) and the expected time of its rounds.
struct TileChoice {
  int mb, nb;
  TailPlan tail;
  double rounds_us;
};
static TileChoice choose_tile(int64_t M, int64_t N, int64_t K, bool row_scales, bool accumulate, const TailPlan& tail) {
  Width w = pick_width(M, N, tail, false);
  Tile t = pick_tile(M, N, K, w, tail, row_scales, false);
  const double us = w.rounds * (9.2 + static_cast<double>(K) * (w.tiles >= kCUs ? 0.0186 : 0.0159)) * (K > 1536 && K <= 4096 ? t.gain : 1.0);
  if (accumulate && K < 1024) {
    w = pick_width(M, N, tail, true);
    t = pick_tile(M, N, K, w, tail, row_scales, true);
  }
  return TileChoice{t.mb, t.nb, t.nb == 8 ? tail : TailPlan{0, 1}, us};
}
// The split is chosen if the workspace has the room for its partial tiles; otherwise the last round is an ordinary one.
static TileChoice choose_tile(int64_t M, int64_t N, int64_t K, bool row_scales, bool accumulate, size_t room_for_partials) {
  const TileChoice c = choose_tile(M, N, K, row_scales, accumulate, plan_tail(M, N, K));
  return partial_bytes(c.tail) <= room_for_partials ? c : choose_tile(M, N, K, row_scales, accumulate, TailPlan{0, 1});
}

// Enough for every way in which the operands may come; a call may use less (plan_two_pass).
size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  size_t partials = 0;
  for (const bool row_scales : {false, true}) partials = std::max(partials, partial_bytes(choose_tile(M, N, K, row_scales, false, SIZE_MAX).tail));
  return operand_bytes(M, N, K) + partials;
}

// What a call does: one answer for the estimate, the room asked of the workspace and the launch.
// Expected time: what is still to decode (codes and scales in, FP16 out) at 5.0 TB/s, then rounds of 256 tiles at 9.2 us for the result and 15.9 ns
// per k while there are fewer, 18.6 when the chip is full (the clock drops with the matrix pipes busy), times what a larger tile gains where the contraction is more of the
// work than storing the result (4112 x 4368 x 128: 256 x 320 tiles take 0.98 of the best others' time, by fewer rounds 0.8) and not so long that the direct kernel's estimate is stretched
// already (plan_route).  Were it to count from K = 1024 on, 82 of 60000 drawn products would leave the direct kernel for it; time there over that in the larger tiles, FP32 / bf16 / accumulated:
// K up to 1536 (56 of them) 0.97 / 1.05 / 0.91 (11648 x 1328 x 1152 accumulated 53 us / 68), up to 4096 (19) 1.04 / 1.11 / 1.00, above (7) 0.94 / 0.96 / 0.88.  All of it is of a plain result, for all output
// types (see SmallTileCost), and what the choice among the kernels is fitted with; estimates nearer to the measured times of this route took it where the
// direct kernel is up to 20 % faster (18.8 us for 4112 x 4368 x 128, 22.6 here).
TwoPassPlan plan_two_pass(const GemmArgs& g) {
  TwoPassPlan plan{false, HUGE_VAL, 8, 8, 0, 1};
  const int64_t M = g.a.outer, N = g.b.outer;
  if (g.K % TK != 0 || g.K >= (int64_t{1} << 21)) return plan;   // (the kernel's 32-bit byte offsets inside a tile)
  const int64_t rows = (g.a.fp16 ? 0 : M) + (g.b.fp16 ? 0 : N);
  const size_t operands = operand_bytes(rows, 0, g.K);
  if (operands > g.workspace_bytes) return plan;
  const TileChoice c = choose_tile(M, N, g.K, g.a.ts_per_row != 0 || g.b.ts_per_row != 0, g.accumulate, g.workspace_bytes - operands);
  plan.us = 7.4 + static_cast<double>(rows) * static_cast<double>(g.K) * 2.5625 / 5.0e6 + c.rounds_us;
  plan.mb = c.mb;
  plan.nb = c.nb;
  plan.tail = c.tail.tail;
  plan.splits = c.tail.splits;
  // (With both operands decoded beforehand and no round split nothing is needed of the workspace.)
  const bool room = operands + partial_bytes(c.tail) == 0 || (g.workspace && reinterpret_cast<uintptr_t>(g.workspace) % 256 == 0);
  plan.usable = room && reinterpret_cast<uintptr_t>(g.a.fp16) % 16 == 0 && reinterpret_cast<uintptr_t>(g.b.fp16) % 16 == 0 &&
                reinterpret_cast<uintptr_t>(g.a.codes) % 16 == 0 && reinterpret_cast<uintptr_t>(g.b.codes) % 16 == 0 &&
                reinterpret_cast<uintptr_t>(g.a.scales) % 4 == 0 && reinterpret_cast<uintptr_t>(g.b.scales) % 4 == 0;
  return plan;
}

#define NVFP4_LAUNCH_F16(BF16, ROWSCALES, SPLIT, MB, NB)                                                              \
  do {                                                                                                            \
    static PerDeviceOnce once;                                                                                    \
    constexpr int lds_bytes = kStages * stage_bytes(MB, NB);                                                      \
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&gemm_f16_kernel<BF16, ROWSCALES, SPLIT, MB, NB>), lds_bytes, once); \
    if (e != hipSuccess) return e;                                                                                \
    hipLaunchKernelGGL((gemm_f16_kernel<BF16, ROWSCALES, SPLIT, MB, NB>), dim3(wgs), dim3(kThreads), lds_bytes, s, a16, b16, \
                       g.a.outer, g.b.outer, g.K, g.a.ts, g.b.ts, g.d, g.ldd, g.accumulate, tiles_m, tiles_n,     \
                       tile_begin, tile_count, k_splits, partials, g.a.ts_per_row != 0, g.b.ts_per_row != 0);      \
  } while (0)

// Tiles [tile_begin, tile_begin + tile_count); k_splits > 1: each shared by that many workgroups, summed by a second launch.
template <int kMB, int kNB>
static hipError_t launch_f16(bool bf16_out, const _Float16* a16, const _Float16* b16, const GemmArgs& g, int tiles_m,
                             int tiles_n, int tile_begin, int tile_count, int k_splits, float* partials, hipStream_t s) {
  // More whole tiles than CUs: one workgroup per CU, each running its tiles as one stream of K steps.
  unsigned wgs = static_cast<unsigned>(tile_count) * static_cast<unsigned>(k_splits);
  if (k_splits == 1 && g.K / TK >= 2 && wgs > static_cast<unsigned>(kCUs)) wgs = kCUs;
  const bool row_scales = g.a.ts_per_row != 0 || g.b.ts_per_row != 0;
  if (k_splits > 1) {
    NVFP4_LAUNCH_F16(false, false, true, 8, 8);
    const dim3 grid(static_cast<unsigned>(tile_count) * 32);   // tile, 128 x 128 block, 16 rows
#define NVFP4_LAUNCH_SUM(BF16, ROWSCALES)                                                                              \
  hipLaunchKernelGGL((splitk_sum_kernel<BF16, ROWSCALES>), grid, dim3(64), 0, s, partials, k_splits, g.a.outer, g.b.outer, \
                     g.a.ts, g.b.ts, g.d, g.ldd, g.accumulate, tiles_m, tiles_n, tile_begin, g.a.ts_per_row != 0,      \
                     g.b.ts_per_row != 0)
    if (bf16_out) {
      if (row_scales) NVFP4_LAUNCH_SUM(true, true); else NVFP4_LAUNCH_SUM(true, false);
    } else {
      if (row_scales) NVFP4_LAUNCH_SUM(false, true); else NVFP4_LAUNCH_SUM(false, false);
    }
#undef NVFP4_LAUNCH_SUM
  } else if (row_scales) {
    if constexpr (kMB == 8) {
      if (bf16_out) NVFP4_LAUNCH_F16(true, true, false, kMB, kNB); else NVFP4_LAUNCH_F16(false, true, false, kMB, kNB);
    } else {
      return hipErrorInvalidValue;   // (pick_tile offers none)
    }
  } else {
    if (bf16_out) NVFP4_LAUNCH_F16(true, false, false, kMB, kNB); else NVFP4_LAUNCH_F16(false, false, false, kMB, kNB);
  }
  return hipGetLastError();
}
#undef NVFP4_LAUNCH_F16

// Grid of the decode pass for `blocks` 16-row blocks: a workgroup per block and kDecodeK elements of K.  False
// if that is more than a grid can hold (operands beyond 2^44 elements).
static bool decode_grid(int64_t blocks, int64_t K, dim3* grid) {
  const int64_t n = blocks * ((K + kDecodeK - 1) / kDecodeK);
  if (n > 0x7fffffff) return false;
  *grid = dim3(static_cast<unsigned>(n));
  return true;
}

hipError_t launch_predecode(const Operand& op, int64_t K, void* fp16_out, hipStream_t s) {
  dim3 grid;
  if (!decode_grid(op.outer / 16, K, &grid)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(decode_f16_kernel, grid, dim3(256), 0, s, op.codes, op.scales,
                     static_cast<int>(op.outer / 16), static_cast<_Float16*>(fp16_out), op.codes, op.scales, 0,
                     static_cast<_Float16*>(fp16_out), K);
  return hipGetLastError();
}

// Every tile in one launch of the kernel with tiles of 32 kMB x 32 kNB.
template <int kMB, int kNB>
static hipError_t launch_all(const GemmArgs& g, const _Float16* a16, const _Float16* b16, hipStream_t s) {
  const int tiles_m = static_cast<int>((g.a.outer + 32 * kMB - 1) / (32 * kMB)), tiles_n = static_cast<int>((g.b.outer + 32 * kNB - 1) / (32 * kNB));
  return launch_f16<kMB, kNB>(g.out_bf16, a16, b16, g, tiles_m, tiles_n, 0, tiles_m * tiles_n, 1, nullptr, s);
}

hipError_t launch_gemm_two_pass(const GemmArgs& g, const TwoPassPlan& plan, hipStream_t s) {
  const int64_t M = g.a.outer, N = g.b.outer, K = g.K;
  // Workspace: [A as FP16 unless decoded beforehand][B likewise][partial tiles]
  char* ws = static_cast<char*>(g.workspace);
  const int64_t rows_a = g.a.fp16 ? 0 : M, rows_b = g.b.fp16 ? 0 : N;
  _Float16* a_ws = reinterpret_cast<_Float16*>(ws);
  _Float16* b_ws = a_ws + rows_a * K;
  const _Float16* a16 = g.a.fp16 ? static_cast<const _Float16*>(g.a.fp16) : a_ws;
  const _Float16* b16 = g.b.fp16 ? static_cast<const _Float16*>(g.b.fp16) : b_ws;
  float* partials = reinterpret_cast<float*>(ws + operand_bytes(rows_a, rows_b, K));
  // One launch decodes what is still to decode.
  if (rows_a + rows_b > 0) {
    dim3 grid;
    if (!decode_grid((rows_a + rows_b) / 16, K, &grid)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(decode_f16_kernel, grid, dim3(256), 0, s, g.a.codes, g.a.scales, static_cast<int>(rows_a / 16), a_ws,
                       g.b.codes, g.b.scales, static_cast<int>(rows_b / 16), b_ws, K);
  }
  if (plan.mb == 10) return launch_all<10, 10>(g, a16, b16, s);
  switch (plan.nb) {
    case 10: return launch_all<8, 10>(g, a16, b16, s);
    case 7: return launch_all<8, 7>(g, a16, b16, s);
    case 6: return launch_all<8, 6>(g, a16, b16, s);
    case 5: return launch_all<8, 5>(g, a16, b16, s);
    default: break;
  }
  const int tiles_m = static_cast<int>((M + TM - 1) / TM), tiles_n = static_cast<int>((N + TN - 1) / TN);
  const int tiles = tiles_m * tiles_n;
  // One 256x256 tile keeps one CU busy (its LDS fits one workgroup).  Whole rounds of kCUs tiles
  // run as they are; a last partial round that fills at most half the chip is split along K.
  const int full = tiles - plan.tail;
  hipError_t e = hipSuccess;
  if (full > 0) e = launch_f16<8, 8>(g.out_bf16, a16, b16, g, tiles_m, tiles_n, 0, full, 1, nullptr, s);
  if (e == hipSuccess && plan.tail > 0)
    e = launch_f16<8, 8>(g.out_bf16, a16, b16, g, tiles_m, tiles_n, full, plan.tail, plan.splits, partials, s);
  return e;
}

}  // namespace nvfp4
