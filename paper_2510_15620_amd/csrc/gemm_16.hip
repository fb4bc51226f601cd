// 16-bit-operand layer contractions on the gfx950 matrix cores (paper Sec. 2.2: the reranker's latency is
// dominated by the matrix multiplications of its transformer blocks).
//
// C = A W^T, A [M,K] and W [N,K] row-major, both bf16 or both IEEE half (K-contiguous, which is what
// the MFMA operand registers want: 8 consecutive k per lane), fp32 accumulation in
// v_mfma_f32_16x16x32_{bf16,f16}.
//
// Workgroup tile BM x BN x 64, WM x WN wavefronts, each owning a (BM/WM) x (BN/WN) block of the accumulator.  The
// large-launch shape is 256 x 256 with 2 x 2 wavefronts (one per SIMD, 128 x 128 each,
// 256 accumulator registers in AGPRs); launches with few tiles per compute unit take one of seven smaller tiles
// down to 32 x 32 (see the choice at the launcher).  A and W tiles are staged in LDS (a ring of S stages, 256 x 256: three
// of A and two of W; 16-byte chunks XOR-swizzled by row so that the 16-row operand reads spread over the banks) by direct
// global->LDS loads, which need no staging registers.  Every K loop is generated text (gen_gemm_kloop.py), because its waits count loads
// and fragment reads exactly; rows beyond the matrix are clamped in the load offsets, so edge tiles run the same loop.
//
// Epilogues: plain store (bf16 or fp32), residual add into the fp32 stream, and SwiGLU, where the B tile is
// made of BN/2 gate rows and the BN/2 matching up rows so that a lane holds g and u of one element.
//
// Workgroup ids are remapped so that each XCD (ids are dealt round-robin over the 8 XCDs) owns a
// contiguous range of tiles, walked in groups of 4 or 8 row-tiles, to keep the operand panels in its L2.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "gemm_16_kloop.inc"

namespace prism {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
static constexpr int BK = 64;            // K-slice per stage (elements)
static constexpr int kChunks = BK / 8;   // 16-byte chunks per tile row

// LDS serves a 16-byte read of 16 consecutive lanes per cycle out of 64 banks; with 128-byte rows the bank
// half is the row's parity, so the chunk is rotated by bits 1..3 of the row.
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

#define PRISM_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define PRISM_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

// silu(g) * u in fp32, rounded to 16 bits by its callers.  The division is correctly rounded: a product with the reciprocal
// instruction takes half of this epilogue's arithmetic away (13.8 -> 9.2 thousand cycles of a 256 x 256 tile) and no time where the
// chip is full and at its power limit (24576 x 24576 x 4096: 3350 us, with the division 3337), but is off by
// an ulp more and returns 0 where 1 + e^-g exceeds 2^126, values that bf16 still holds.
__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

// LDS bytes of a tile's operand stages
template <int BM, int BN, int S> constexpr int stage_bytes() { return ((BM == 256 ? 3 : S) * BM + S * BN) * BK * 2; }

template <typename OT, int BM, int BN, int WM, int WN, int EPI, int S>
__global__ __launch_bounds__(WM *WN * 64, (stage_bytes<BM, BN, S>() > 81920 ? 1 : 2)) void gemm_16_kernel(const OT *__restrict__ A,
                                                               const OT *__restrict__ W, void *__restrict__ out_,
                                                               int M, int N, int K, int nM, int nN, QkvEpilogue qe) {
  constexpr int NW = WM * WN;
  constexpr bool kHeads = EPI == kEpiQkv;
  constexpr int WMT = BM / WM, WNT = BN / WN;      // wave tile
  constexpr int TM = WMT / 16, TN = WNT / 16;      // 16 x 16 accumulator tiles per wave
  // one direct-to-LDS instruction of a wave moves 64 x 16 B = 8 tile rows
  constexpr int A_ITERS = BM / 8 / NW, B_ITERS = BN / 8 / NW;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile/waves mismatch");
  static_assert(EPI != PRISM_EPI_SWIGLU || TN % 2 == 0, "SwiGLU pairs gate and up tiles");
  static_assert(TM * TN * 4 <= 256, "accumulator registers");
  extern __shared__ __align__(16) unsigned char smem[];
  static_assert(BM != 256 || S == 2, "the 256 x 256 loop has three stages of A and two of W");
  OT *lA = reinterpret_cast<OT *>(smem);                     // [S, or 3 if BM == 256][BM][BK]
  OT *lB = lA + (BM == 256 ? 3 : S) * BM * BK;               // [S][BN][BK]

  // ---- tile mapping: XCD-contiguous ranges, grouped walk ----
  const int n_tiles = nM * nN;
  int bid = blockIdx.x;
  {
    const int per = (n_tiles + 7) / 8, x = bid % 8, r = bid / 8;
    // XCD x owns logical ids [x*per, ...); ids beyond n_tiles idle
    bid = x * per + r;
    if (r >= per || bid >= n_tiles) return;
  }
  // 256 x 256: an XCD runs 32 tiles at a time, 4 row-tiles x 8 column-tiles of them or 8 x 4 - the same operand bytes - but 4 is
  // 3 % faster at 24576 x 24576 x 4096 (1364 -> 1410 TFLOP/s; 3, 5, 6, 8, 16: 1-4 % slower, on some chips 6 %), and 4 % than 8
  // at 32768 x 4096 x 12288
  constexpr int GM = BM == 256 || EPI == PRISM_EPI_RESIDUAL ? 4 : 8;
  const int group = bid / (GM * nN), first_m = group * GM;
  const int gsz = (nM - first_m) < GM ? (nM - first_m) : GM;
  const int tile_m = first_m + (bid % (GM * nN)) % gsz, tile_n = (bid % (GM * nN)) / gsz;
  const int m0 = tile_m * BM;
  const int F = EPI == PRISM_EPI_SWIGLU ? N / 2 : N;         // output columns
  constexpr int BNO = EPI == PRISM_EPI_SWIGLU ? BN / 2 : BN; // output columns per tile
  const int n0 = tile_n * (EPI == PRISM_EPI_SWIGLU ? BN / 2 : BN);

  // read from a lane, so that what follows from the wave's place stays in scalar registers
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- global -> LDS staging without registers (global_load_lds_dwordx4).  Instruction j of wave w
  //      fills tile rows (w * ITERS + j) * 8 .. + 8, lane l landing at row l / 8, chunk slot l % 8.
  //      The XOR swizzle is applied on the source side: slot p of row r receives chunk swz(r, p).
  const int lrow = lane >> 3;
  // byte offsets from the tile's first row of A / W, rows beyond the matrix clamped; four loads share one destination register and
  // carry 0, 1, 2, 3 KiB in the instruction, which shifts the source too: taken off here, with 4 KiB in hand (kBias)
  constexpr uint32_t kBias = 4096;
  uint32_t gA[A_ITERS], gB[B_ITERS];
#pragma unroll
  for (int j = 0; j < A_ITERS; ++j) {
    const int row = (wave * A_ITERS + j) * 8 + lrow;
    const int r = m0 + row < M ? row : M - 1 - m0;
    gA[j] = ((uint32_t)r * (uint32_t)K + swz(row, lane & 7) * 8) * 2u + kBias - j % 4 * 1024u;
  }
#pragma unroll
  for (int j = 0; j < B_ITERS; ++j) {
    const int row = (wave * B_ITERS + j) * 8 + lrow;
    const int half = EPI == PRISM_EPI_SWIGLU ? row / (BN / 2) : 0, rr = row - half * (BN / 2);   // gate rows, then up rows
    const int r = (n0 + rr < F ? rr : F - 1 - n0) + half * F;
    gB[j] = ((uint32_t)r * (uint32_t)K + swz(row, lane & 7) * 8) * 2u + kBias - j % 4 * 1024u;
  }
  // ---- LDS rows this lane reads as MFMA operands: row (A) and first column (B) of its first fragment; it feeds 8 of the
  //      32 k of one of 16 rows to an MFMA
  const int frow = lane & 15, kpart = lane >> 4;
  const int rA0 = wm * WMT + frow, rB0 = wn * (EPI == PRISM_EPI_SWIGLU ? WNT / 2 : WNT) + frow;

  // accumulator tile (i, j) is a[4 t .. 4 t + 3], t = i TN + j: four tiles to an operand of the K loop, which clears them
  f32x16 acc[(TM * TN + 3) / 4];

  const int nk = K / BK;

  // ---- epilogue geometry (see the epilogue): everything it reads or writes goes along the rows, 16 bytes per lane.
  //      Residual epilogue: the old values of a block of 32 rows (16 in the smallest tiles) are requested one block ahead, the first block's
  //      before the K loop where registers are left (tiles below 256; the big tile spills).  The same for what the q/k/v
  //      epilogue reads by row: a small tile's loop is a few microseconds, and each dependent load behind it about one.
  //      (28 layers of the 0.6B shape on 391 rows, with the same in the RMSNorm: 2749 -> 2687 us.)
  constexpr bool kEarly = BM < 256;
  constexpr bool kF32Out = EPI == PRISM_EPI_RESIDUAL || EPI == PRISM_EPI_STORE_F32;
  constexpr int ES = kF32Out ? 4 : 2;                               // bytes per output element
  constexpr int OUTW = EPI == PRISM_EPI_SWIGLU ? WNT / 2 : WNT;    // output columns of the wave
  constexpr int RB = OUTW * ES, CPR = RB / 16;                      // bytes / 16-byte chunks per staged row
  constexpr int BR = WMT < 32 ? WMT : 32, RPB = BR / 16;            // rows of a block, of those in a lane
  constexpr int NBLK = WMT / BR;                                    // blocks of the wave
  constexpr int NR = 1024 / RB < BR ? 1024 / RB : BR, NI = BR / NR; // rows per instruction, instructions per block
  // lane -> (row within an instruction, chunk); 16 rows of 16 16-bit columns are less than an instruction moves: half the lanes idle
  const int f_row = lane / CPR % NR, f_chunk = lane % CPR;
  const bool f_on = lane / CPR < NR;
  const bool full_n = n0 + BNO <= F && (F * ES) % 16 == 0;
  f32x4 old[2][EPI == PRISM_EPI_RESIDUAL ? NI : 1];
  // An access goes to a wave-uniform address (scalar) plus a lane offset that stays the same: multiplying rows by the pitch per
  // lane and access took a third of the epilogue's vector time.
  const int64_t out_pitch = (int64_t)F * ES;                        // bytes
  const unsigned f_off = (unsigned)f_row * (unsigned)out_pitch + (unsigned)f_chunk * 16u;   // < 32 rows: far below 4 GiB
  unsigned char *const out_w = reinterpret_cast<unsigned char *>(out_) + (int64_t)(m0 + wm * WMT) * out_pitch + (int64_t)(n0 + wn * OUTW) * ES;
  const int rows_left = M - m0 - wm * WMT;                          // of the wave's rows inside the matrix
  const int64_t out_step = NR * out_pitch;
  const unsigned char *old_at = out_w;                              // steps along with the loads
  // (whole: every row is inside the matrix, no guard per access)
  auto load_old = [&](int i, auto whole) __attribute__((always_inline)) {
    if constexpr (EPI == PRISM_EPI_RESIDUAL) {
#pragma unroll
      for (int rr = 0; rr < NI; ++rr) {
        const int r = i * BR + rr * NR;
        if (whole || r + f_row < rows_left) old[i & 1][rr] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(old_at + f_off));
        old_at += out_step;
      }
    }
  };


  int row_in[kHeads ? TM : 1];                                // q, k heads: positions; v heads: V^T columns
  auto load_rows = [&]() __attribute__((always_inline)) {
    if constexpr (kHeads) {
      const int32_t *src = ((n0 + wn * WNT) >> 7) < qe.nq + qe.nkv ? qe.pos : qe.vt_col;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m0 + wm * WMT + i * 16 + frow;
        row_in[i] = src[row < M ? row : M - 1];
      }
    }
  };
  if constexpr (kEarly) {
    if constexpr (kHeads) load_rows();
    else if (full_n) load_old(0, std::false_type{});
  }

  // ---- epilogue.  The W fragment was the instruction's first operand, so the 16 x 16 accumulator tile (i, j) is transposed:
  //      a lane holds ONE row of A, 16 i + lane % 16, and 4 consecutive output columns 16 j + 4 (lane / 16) + q, q = 0..3.
  //      Written straight from that layout, one store instruction touches 32 rows with 16-32 bytes in each, and
  //      the number of cache lines an instruction touches - not the bytes - is what the memory path charges for
  //      (measured: 12-29 us per 256 x 256 tile, a tenth to a fifth of the tile's time).  So every block of rows goes
  //      through LDS, which is free once the K loop is done: lanes write their row's values, then read back 16 bytes
  //      each along the rows, so that an instruction reads or writes whole lines (2-8 complete rows of the wave's
  //      columns).  LDS requests of one wave are served in order, so no barrier is needed between the two phases.
  auto epilogue = [&]() __attribute__((always_inline)) {
  // Accumulator element (i, j, q), fetched from its accumulation register when it is needed: behind the hand-scheduled
  // loop all 256 of them sit in AGPRs, and read as plain values the compiler would copy the whole set into vector
  // registers at once, leaving none for the epilogue's own arithmetic.
  // (The compiler does not look inside these statements, so the wait between a matrix instruction and the first read
  // of its result is spelled out: every accumulator tile passes through an empty statement, which puts all matrix
  // instructions before it, then 32 idle cycles - more than the deepest instruction needs to retire.  All of these are
  // volatile, which keeps them in this order.)
#pragma unroll
  for (int t = 0; t < (TM * TN + 3) / 4; ++t) asm volatile("" : "+a"(acc[t]));
  asm volatile("s_nop 15\n\ts_nop 15");
  auto AC = [&](int i, int j, int q) __attribute__((always_inline)) {
    float r;
    const int t = i * TN + j;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(acc[t / 4][t % 4 * 4 + q]));
    return r;
  };
  __syncthreads();              // every wave's operand loads have landed and nobody reads operands any more
  constexpr int SWZ = CPR >= 16 ? 15 : CPR - 1;                     // chunk rotation by row: spreads a column of 16-byte
                                                                    // writes (one per row) over the banks
  // the lane's place again, from the thread index: kept over the loop, one of these ends in scratch memory, and its reload waits for
  // every old value requested before it
  unsigned again = threadIdx.x;
  asm volatile("" : "+v"(again));
  const int e_row = again & 15, e_col = (again & 63) >> 4 << 2;     // row and column in an accumulator tile
  static_assert(NR * RB == 1024 || !kF32Out, "the residual's accesses have no idle lanes");
  static_assert(BR * RB <= stage_bytes<BM, BN, S>() / NW, "staging block must fit the wave's share of LDS");
  unsigned char *stg = smem + wave * (stage_bytes<BM, BN, S>() / NW);
  // values for columns n .. n + 3 (n a multiple of 4, within the wave's columns) of staged row m
  auto put32 = [&](int m, int n, const f32x4 &v) __attribute__((always_inline)) {
    *reinterpret_cast<f32x4 *>(stg + m * RB + (((n >> 2) ^ (m & SWZ)) << 4)) = v;
  };
  auto put16 = [&](int m, int n, const typename Mfma<OT>::vec4 &v) __attribute__((always_inline)) {
    *reinterpret_cast<typename Mfma<OT>::vec4 *>(stg + m * RB + (((n >> 3) ^ (m & SWZ)) << 4) + (n & 4) * 2) = v;
  };
  auto staged = [&](int rr) __attribute__((always_inline)) {
    const int r = rr * NR + f_row;
    return *reinterpret_cast<const uint4 *>(stg + r * RB + ((f_chunk ^ (r & SWZ)) << 4));
  };
  // Flushes the staged block i of the wave's rows to a row-major destination (wave-uniform address of the wave's first row and
  // column, row pitch, the lane's offset).
  auto flush_store = [&](unsigned char *dst, int64_t pitch, unsigned off, int i) __attribute__((always_inline)) {
    dst += (int64_t)i * BR * pitch;
#pragma unroll
    for (int rr = 0; rr < NI; ++rr) {
      const uint4 v = staged(rr);
      if (f_on && i * BR + rr * NR + f_row < rows_left) __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t *>(dst + off));
      dst += NR * pitch;
    }
  };

  if constexpr (kHeads) {
    // The wave's 128 columns are one head.  A row's 128 values sit in the 4 lanes with the same lane % 16; the rotate-half
    // partner of column d is d + 64 = the same register of accumulator tile j + 4, so the per-head RMSNorm
    // (two cross-lane adds), the rotation and the single rounding all happen on the accumulators.  What the memory path
    // charges for is cache lines touched per instruction, so the cos/sin pairs come from the TRANSPOSED table (the 16
    // tokens of a load are consecutive positions of a sequence almost always: four lines per load instead of
    // one or two per lane) and the finished q / k rows go through the staging block like the other epilogues' outputs.
    static_assert(WNT == 128, "one head per wavefront");
    typedef typename Mfma<OT>::vec4 vec4;
    const int head = (n0 + wn * WNT) >> 7;                 // wave-uniform
    if constexpr (!kEarly) load_rows();                    // all rows' at once: one memory latency, not one per block
    if (head < qe.nq + qe.nkv) {
      const OT *gain = reinterpret_cast<const OT *>(head < qe.nq ? qe.q_gain : qe.k_gain);
      vec4 ga[4], gb[4];
      if (qe.qk_norm) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ga[j] = *reinterpret_cast<const vec4 *>(gain + j * 16 + e_col);
          gb[j] = *reinterpret_cast<const vec4 *>(gain + j * 16 + e_col + 64);
        }
      }
      const int64_t pitch = (int64_t)(qe.nq + qe.nkv) * 128 * 2;
      unsigned char *const qk_w = reinterpret_cast<unsigned char *>(qe.QK) + (int64_t)(m0 + wm * WMT) * pitch + (int64_t)head * 128 * 2;
      const unsigned qk_off = (unsigned)f_row * (unsigned)pitch + (unsigned)f_chunk * 16u;
      // (cos, sin) of (pos, d) sits at [d * stride + pos]: a wave-uniform base per column plus one 32-bit lane offset (in bytes, or
      // the compiler cannot rule out a carry and adds 64-bit addresses per lane).
      // The pairs of block i + 1 are requested before block i is worked on, so the tile pays the memory latency once,
      // not once per block.
      unsigned lane_off[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) lane_off[i] = ((unsigned)(e_col) * (unsigned)qe.rope_stride + (unsigned)row_in[i]) * 8u;
      float2 cs[2][RPB][4][4];
      auto load_cs = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < RPB; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const char *col = reinterpret_cast<const char *>(qe.rope_tab_t + (int64_t)(j * 16 + q) * qe.rope_stride);
              cs[b & 1][h][j][q] = *reinterpret_cast<const float2 *>(col + lane_off[b * RPB + h]);
            }
      };
      load_cs(0);
#pragma unroll
      for (int b = 0; b < NBLK; ++b) {
        if (b + 1 < NBLK) load_cs(b + 1);
        float r[RPB];
#pragma unroll
        for (int h = 0; h < RPB; ++h) {
          r[h] = 1.f;
          if (qe.qk_norm) {
            // the finishing kernel's order of the sum of squares: column pairs (d, d + 64), then halving over the bits of d, 32 first
            const int i = b * RPB + h;
            float p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              auto pair = [&](int j) __attribute__((always_inline)) {
                const float x = AC(i, j, q), y = AC(i, j + 4, q);
                return __builtin_fmaf(x, x, y * y);
              };
              p[q] = sum_xor16(sum_xor32((pair(0) + pair(2)) + (pair(1) + pair(3))));
            }
            r[h] = 1.0f / sqrtf(((p[0] + p[2]) + (p[1] + p[3])) / 128.f + qe.eps);
          }
        }
#pragma unroll
        for (int h = 0; h < RPB; ++h)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            vec4 lo, hi;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float2 c = cs[b & 1][h][j][q];
              float x = AC(b * RPB + h, j, q), y = AC(b * RPB + h, j + 4, q);
              if (qe.qk_norm) {
                x = x * r[h] * to_f32(ga[j][q]);
                y = y * r[h] * to_f32(gb[j][q]);
              }
              lo[q] = from_f32<OT>(__builtin_fmaf(x, c.x, -(y * c.y)));
              hi[q] = from_f32<OT>(__builtin_fmaf(y, c.x, x * c.y));
            }
            put16(h * 16 + e_row, j * 16 + e_col, lo);
            put16(h * 16 + e_row, j * 16 + e_col + 64, hi);
          }
        flush_store(qk_w, pitch, qk_off, b);
      }
    } else {
      // v head: rounded to the operand type, stored as half, transposed (16 consecutive tokens of one d are contiguous)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (m0 + wm * WMT + i * 16 + e_row >= M) continue;
        f16 *vt = reinterpret_cast<f16 *>(qe.Vt) + ((int64_t)(head - qe.nq - qe.nkv) * 128 + e_col) * qe.vt_stride + row_in[i];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            vt[(int64_t)(j * 16 + q) * qe.vt_stride] = from_f32<f16>(to_f32(from_f32<OT>(AC(i, j, q))));
      }
    }
    return;
  }

  if (EPI == PRISM_EPI_RESIDUAL && full_n) {
    // read-modify-write of the fp32 stream, whole lines per instruction; the loads of the next block are requested
    // before this block is staged, so the tile pays the memory latency once, not per block
    auto residual = [&](auto whole) __attribute__((always_inline)) {
      if constexpr (!kEarly) load_old(0, whole);
      int64_t new_at = 0;
      asm volatile("" : "+s"(new_at));       // a chain of its own: 64 addresses shared with the loads would not fit the scalar registers
#pragma unroll
      for (int b = 0; b < NBLK; ++b) {
        if (b + 1 < NBLK) load_old(b + 1, whole);
#pragma unroll
        for (int h = 0; h < RPB; ++h)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = AC(b * RPB + h, j, q);
            put32(h * 16 + e_row, j * 16 + e_col, v);
          }
#pragma unroll
        for (int rr = 0; rr < NI; ++rr) {
          const int r = b * BR + rr * NR;
          const uint4 u = staged(rr);
          f32x4 v = old[b & 1][rr];
          v[0] += __uint_as_float(u.x); v[1] += __uint_as_float(u.y); v[2] += __uint_as_float(u.z); v[3] += __uint_as_float(u.w);
          if (whole || r + f_row < rows_left) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(out_w + new_at + f_off));
          new_at += out_step;
        }
      }
    };
    if (rows_left >= WMT) residual(std::true_type{});
    else residual(std::false_type{});
    return;
  }
  if (full_n) {
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
#pragma unroll
      for (int h = 0; h < RPB; ++h)
#pragma unroll
        for (int j = 0; j < OUTW / 16; ++j) {
          const int i = b * RPB + h, row = h * 16 + e_row, col = j * 16 + e_col;
          if constexpr (EPI == PRISM_EPI_STORE_F32) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = AC(i, j, q);
            put32(row, col, v);
          } else {
            typename Mfma<OT>::vec4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = from_f32<OT>(EPI == PRISM_EPI_SWIGLU ? silu_mul(AC(i, j, q), AC(i, j + TN / 2, q)) : AC(i, j, q));
            put16(row, col, v);
          }
        }
      flush_store(out_w, out_pitch, f_off, b);
    }
    return;
  }

  // ---- ragged last column tile (N not a multiple of the tile, or rows not 16-byte aligned): element by element
  if constexpr (!kHeads) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < OUTW / 16; ++j)
        for (int q = 0; q < 4; ++q) {
          const int row = m0 + wm * WMT + i * 16 + e_row, col = n0 + wn * OUTW + j * 16 + e_col + q;
          if (row >= M || col >= F) continue;
          if (EPI == PRISM_EPI_SWIGLU) {
            reinterpret_cast<OT *>(out_)[(int64_t)row * F + col] = from_f32<OT>(silu_mul(AC(i, j, q), AC(i, j + TN / 2, q)));
          } else if (EPI == PRISM_EPI_RESIDUAL) {
            reinterpret_cast<float *>(out_)[(int64_t)row * N + col] += AC(i, j, q);
          } else if (EPI == PRISM_EPI_STORE_F32) {
            reinterpret_cast<float *>(out_)[(int64_t)row * N + col] = AC(i, j, q);
          } else {
            reinterpret_cast<OT *>(out_)[(int64_t)row * N + col] = from_f32<OT>(AC(i, j, q));
          }
        }
  }
  };

  const unsigned ldsA = (unsigned)(uintptr_t)PRISM_LDS_PTR(lA), ldsB = (unsigned)(uintptr_t)PRISM_LDS_PTR(lB);
  const unsigned aA0 = ldsA + (unsigned)(rA0 * BK + swz(rA0, kpart) * 8) * 2u;
  const unsigned aB0 = ldsB + (unsigned)(rB0 * BK + swz(rB0, kpart) * 8) * 2u;
  // wave w's load instruction j fills tile rows (w * ITERS + j) * 8 .. + 8 of an operand (1 KiB of LDS)
  const unsigned ldsA_w = __builtin_amdgcn_readfirstlane(ldsA + (unsigned)wave * A_ITERS * 8 * BK * 2);
  const unsigned ldsB_w = __builtin_amdgcn_readfirstlane(ldsB + (unsigned)wave * B_ITERS * 8 * BK * 2);
  const uint64_t baseA = (uint64_t)(uintptr_t)A + (uint64_t)m0 * K * 2 - kBias, baseB = (uint64_t)(uintptr_t)W + (uint64_t)n0 * K * 2 - kBias;
  // the upper half of the wave's columns: SwiGLU's are the up rows, half a tile further (the swizzle repeats every 16 rows)
  const unsigned aB1 = aB0 + (unsigned)((EPI == PRISM_EPI_SWIGLU ? BN / 2 : WNT / 2) * BK) * 2u;
#define PRISM_ACC1 "={a[0:15]}"(acc[0])
#define PRISM_ACC2 PRISM_ACC1, "={a[16:31]}"(acc[1])
#define PRISM_ACC4 PRISM_ACC2, "={a[32:47]}"(acc[2]), "={a[48:63]}"(acc[3])
#define PRISM_ACC16                                                                                                               \
  PRISM_ACC4, "={a[64:79]}"(acc[4]), "={a[80:95]}"(acc[5]), "={a[96:111]}"(acc[6]), "={a[112:127]}"(acc[7]),                        \
      "={a[128:143]}"(acc[8]), "={a[144:159]}"(acc[9]), "={a[160:175]}"(acc[10]), "={a[176:191]}"(acc[11]), "={a[192:207]}"(acc[12]), \
      "={a[208:223]}"(acc[13]), "={a[224:239]}"(acc[14]), "={a[240:255]}"(acc[15])
  // (offsets of loads that a tile does not have are never named by its loop)
#define PRISM_AB(j) [ga##j] "v"(gA[j < A_ITERS ? j : 0]), [gb##j] "v"(gB[j < B_ITERS ? j : 0])
#define PRISM_RUN_TY(LOOP, CLOBBERS, ...)                                                                                       \
  asm volatile(LOOP : __VA_ARGS__                                                                                              \
               : [aa] "v"(aA0), [ab] "v"(aB0), [ab2] "v"(aB1), PRISM_AB(0), PRISM_AB(1), PRISM_AB(2), PRISM_AB(3), PRISM_AB(4), \
                 PRISM_AB(5), PRISM_AB(6), PRISM_AB(7), [la] "s"(ldsA_w), [lb] "s"(ldsB_w), [pa] "s"(baseA), [pb] "s"(baseB),   \
                 [nk] "s"(nk)                                                                                                  \
               : CLOBBERS)
#define PRISM_RUN(NAME, ...)                                                                                                    \
  do {                                                                                                                         \
    if constexpr (Mfma<OT>::kIsF16) PRISM_RUN_TY(PRISM_KLOOP_##NAME("f16"), PRISM_KLOOP_CLOBBERS_##NAME, __VA_ARGS__);          \
    else PRISM_RUN_TY(PRISM_KLOOP_##NAME("bf16"), PRISM_KLOOP_CLOBBERS_##NAME, __VA_ARGS__);                                    \
  } while (0)
  if constexpr (BM == 256) PRISM_RUN(256, PRISM_ACC16);
  else if constexpr (kHeads && BM == 64 && S == 6) PRISM_RUN(64x128_6_HEAD, PRISM_ACC2);
  else if constexpr (kHeads && BM == 64) PRISM_RUN(64x128_3_HEAD, PRISM_ACC2);
  else if constexpr (kHeads && S == 5) PRISM_RUN(128x128_5_HEAD, PRISM_ACC4);
  else if constexpr (kHeads && S == 3) PRISM_RUN(128x128_3_HEAD, PRISM_ACC4);
  else if constexpr (kHeads) PRISM_RUN(128x128_2_HEAD, PRISM_ACC4);
  else if constexpr (BM == 32 && BN == 32) PRISM_RUN(32x32_9, PRISM_ACC1);
  else if constexpr (BM == 64 && BN == 32) PRISM_RUN(64x32_7, PRISM_ACC1);
  else if constexpr (BM == 32 && BN == 64) PRISM_RUN(32x64_4, PRISM_ACC2);
  else if constexpr (BM == 64 && BN == 64) PRISM_RUN(64x64_5, PRISM_ACC1);
  else if constexpr (BM == 128 && BN == 64 && S == 6) PRISM_RUN(128x64_6, PRISM_ACC2);
  else if constexpr (BM == 128 && BN == 64) PRISM_RUN(128x64_3, PRISM_ACC2);
  else if constexpr (S == 5) PRISM_RUN(128x128_5, PRISM_ACC4);
  else if constexpr (S == 4) PRISM_RUN(128x128_4, PRISM_ACC4);
  else PRISM_RUN(128x128_2, PRISM_ACC4);
#undef PRISM_RUN
#undef PRISM_RUN_TY
#undef PRISM_AB
  epilogue();
}

bool gemm_16_supported(int epilogue, int N, int K) {
  if (K <= 0 || K % BK != 0 || N <= 0) return false;
  if (epilogue == PRISM_EPI_SWIGLU && N % 2 != 0) return false;
  return epilogue >= PRISM_EPI_STORE && epilogue <= PRISM_EPI_STORE_F32;
}

template <typename OT, int BM, int BN, int WM, int WN, int EPI, int S>
static int launch_cfg(const OT *A, const OT *W, void *out, int M, int N, int K, hipStream_t s,
                      const QkvEpilogue &qe = QkvEpilogue{}) {
  constexpr size_t lds = stage_bytes<BM, BN, S>();
  auto kern = gemm_16_kernel<OT, BM, BN, WM, WN, EPI, S>;
  // the attribute is per function: set once per process, also when several contexts launch from different threads
  static std::once_flag attr_once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  PRISM_HIP(attr_rc);
  const int ncols = EPI == PRISM_EPI_SWIGLU ? N / 2 : N, bn_out = EPI == PRISM_EPI_SWIGLU ? BN / 2 : BN;
  const int nM = cdiv(M, BM), nN = cdiv(ncols, bn_out);
  const int grid = cdiv((int64_t)nM * nN, 8) * 8;
  kern<<<grid, WM * WN * 64, lds, s>>>(A, W, out, M, N, K, nM, nN, qe);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ---- which tile a launch uses -----------------------------------------------------------------------------------------
// Rows are independent, columns are independent, and every tile size gives an element the same bits (one accumulator, K in
// order), so the choice is made on time alone.  A launch deals its tiles over 256 compute units; n = tiles per unit, rounded
// up.  A tile's time is its K slices plus a fixed part (dispatch, first slice, epilogue), and a slice's time depends on how
// many tiles share the unit: alone it is a chain of latencies, together the matrix pipes and LDS.  The constants were fit to loops
// on 32x32x16 MFMAs with operands that stay in the caches (256 x 256: to those of today); with weights from memory and the loops of
// today they are off by 11-23 % (root mean square) per tile, 256 x 256 by 30 % where the chip is not full, but what counts is the pick: on
// 265 launches (N 1024-24576, K 1024-12288, 1 to 20000 rows, three epilogues) it is on average 0.6 % above the best tile and ring.  The
// costs are of the shallow rings (deep_ring, below, only says which ring the picked tile runs on), so the worst picks stand beside a 128 x 64
// tile on its deeper one: 150 x 6144 x 2560 stored 21.7 us on 32 x 64, 16.8 there, 150 x 6144 x 4096 28.4 and 23.1; next 64 x 19456 x 2560 with
// SwiGLU, 35.1 on 64 x 64 and 30.4 on 128 x 128.  Examples, us with weights from memory, 32x32x16 loops -> now: 100 x 4096 x 12288
// 38.8 -> 38.7 (64 x 32), 391 x 1024 x 3072 10.2 -> 10.0 (64 x 32), 33 x 2560 x 9728 19.3 -> 18.5 (32 x 32), 777 x 6144 x 1024 with SwiGLU
// 19.7 -> 19.1 (128 x 128), 3699 x 1024 x 3072 34.0 -> 32.8 (128 x 128, four stages).
// (256 x 256: on chips of different speed a slice takes 1.34-1.7 us, the fixed part 11 us with SwiGLU and 17 with a residual or a
// head; 1024 x 24576 x 4096 with SwiGLU 233 us on 128 x 128 tiles, 203 on these; 1536 x 6144 x 4096 with heads 103 and 90.)
struct TileCost {
  int bm, bn, occ;              // tile, workgroups that share a compute unit
  float alone, shared, fixed;   // us per 64-deep slice: one workgroup on the unit; per workgroup when occ of them share it; us per tile
};
enum { kTile256, kTile128, kTile128Deep, kTile128x64, kTile64, kTile32x64, kTile64x32, kTile32, kTileKinds };
static constexpr TileCost kTileCost[kTileKinds] = {
    {256, 256, 1, 1.45f, 1.45f, 9.2f}, {128, 128, 2, 0.72f, 0.50f, 4.5f}, {128, 128, 1, 0.52f, 0.52f, 3.4f}, {128, 64, 2, 0.34f, 0.36f, 2.3f},
    {64, 64, 2, 0.204f, 0.204f, 2.1f}, {32, 64, 3, 0.176f, 0.149f, 2.4f}, {64, 32, 1, 0.128f, 0.128f, 2.3f}, {32, 32, 2, 0.106f, 0.083f, 2.6f}};
// The fused q/k/v projection: tiles whose waves own whole heads (the same: off by 9-18 %, 256 x 256 by 25 %; the pick is the best tile and
// ring of 33 of 34 launches of 1 to 12000 rows, 2 % off on one).  Its epilogue is longer: two dependent loads (position, rotation)
// and the per-head arithmetic.  391 x 4096 x 1024: 11 us, where the projection to fp32 and its two finishing kernels took 48;
// 777 x 6144 x 4096: 62.
enum { kHead256, kHead128, kHead128Deep, kHead64, kHeadKinds };
static constexpr TileCost kHeadCost[kHeadKinds] = {
    {256, 256, 1, 1.40f, 1.40f, 17.f}, {128, 128, 2, 0.70f, 0.55f, 5.5f}, {128, 128, 1, 0.52f, 0.52f, 5.0f}, {64, 128, 2, 0.29f, 0.37f, 5.0f}};

static double tile_cost(const TileCost &t, int64_t M, int64_t ncols, int K, bool glu) {
  const int bn = glu ? t.bn / 2 : t.bn;
  const int64_t tiles = (M + t.bm - 1) / t.bm * ((ncols + bn - 1) / bn), n = (tiles + 255) / 256;
  const int64_t full = n / t.occ, rest = n % t.occ;
  const double slice = full * std::max(t.alone, t.shared * t.occ) + (rest ? std::max(t.alone, t.shared * rest) : 0.f);
  return (K / BK) * slice + (double)((n + t.occ - 1) / t.occ) * t.fixed;
}

// What a launch of M rows runs: rows_big rows (whole 256-row tiles, possibly none) on tile kind 0, the rest on kind `kind`.
struct TilePlan { int rows_big, kind; };
static TilePlan plan_tiles(const TileCost *costs, int kinds, int M, int ncols, int K, bool glu) {
  auto best = [&](int rows, double *cost) {
    int at = 0;
    *cost = tile_cost(costs[0], rows, ncols, K, glu);
    for (int k = 1; k < kinds; ++k) {
      if (glu && costs[k].bn == 32) continue;              // SwiGLU pairs a gate and an up tile in a wave
      const double c = tile_cost(costs[k], rows, ncols, K, glu);
      if (c < *cost) { *cost = c; at = k; }
    }
    return at;
  };
  double whole, rest;
  TilePlan p{0, best(M, &whole)};
  // The last round of big tiles may fill only a few compute units at a whole tile's price: then the row tiles that fill
  // whole rounds go to the big tile and the remaining rows to a second launch with whatever suits them.
  const int nN = cdiv(ncols, glu ? 128 : 256), nM = cdiv(M, 256);
  const int rows_big = (int)std::min<int64_t>(nM, ((int64_t)nM * nN / 256) * 256 / nN) * 256;
  if (rows_big > 0 && rows_big < M) {
    const int kind = best(M - rows_big, &rest);
    if (kind != 0 && tile_cost(costs[0], rows_big, ncols, K, glu) + rest < 0.98 * whole) p = {rows_big, kind};
  }
  return p;
}

// Tiles of 128 rows, and of the heads' 64 x 128, have a second ring of slices that takes a whole compute unit's LDS: two more
// slices in flight (128 x 64 and 64 x 128: 6 stages for 3, 128 x 128: 5 for 4 or 3).  It pays where no unit has a second tile to
// run beside the first (over 256 tiles of 128 x 64: up to 25 % slower) and the loop is long enough for its longer start.  us, weights from
// memory, 128 x 64: 391 x 4096 x 12288 78.7 -> 63.6, 391 x 2560 x 9728 59.5 -> 46.6, 1154 x 1024 x 3072 21.0 -> 17.6, with SwiGLU 200 x
// 6144 x 1024 9.7 -> 9.1; of the 59 launches that the rule takes 4-26 % faster or level, where a residual add of K = 1024, which it leaves out, lost up to
// 14 % (2000 x 1024 x 1024 9.1 -> 10.4).  128 x 128: 1154 x 2560 x 9728 76.1 -> 69.0, 900 x 4096 x 12288 103 -> 93; K = 1024 lost 2-27 %
// (777 x 4096 x 1024 11.8 -> 14.7).  64 x 128 of the heads: 391 x 4096 x 1024 11.4 -> 10.8, 200 x 6144 x 4096 31.1 -> 27.1, 64 x 6144 x 2560 26.6 -> 26.9 (the
// worst).  The gain is that of a last row tile with few rows inside the matrix, whose unit loads less.  Where it is more than half full, 128 x 128
// is level on a long K (SwiGLU 100 x 24576 x 4096 48.1 -> 48.2, 128 x 24576 x 4096 50.3 -> 50.8, residual 1500 x 2560 x 4096 39.7 -> 39.4) and loses up to 6 % on a
// shorter one: residual 3699 x 1024 x 3072 32.8 -> 34.1, 2000 x 1024 x 3072 27.5 -> 29.1, SwiGLU 256 x 16384 x 2048 25.2 -> 26.3, 100 x 19456 x 2560 32.3 -> 32.9, heads
// 896 x 4096 x 2048 23.3 -> 23.5, where SwiGLU of 391 x 8192 x 2048 takes 21.9 -> 21.0 and heads of 777 x 4096 x 2048 21.1 -> 20.1.  128 x 64 with SwiGLU,
// 200 x 8192 x 1024 10.0 -> 9.6, 256 x 8192 x 1024 10.5 -> 10.7, 256 x 5504 x 2048 17.0 -> 16.6.  On weights that the caches hold, which a layer's are not behind
// the layers before it: 128 x 64, 391 x 2560 x 4096 20.9 -> 19.7, but 391 x 4096 x 1024 stored 7.1 -> 7.6; 128 x 128, 777 x 4096 x 4096 31.2 -> 31.9.
// 128 x 128 on all units: from K = 3072 on (916 x 4096 x 3072 of heads 30.8 -> 30.7, x 4096 38.5 -> 36.3, but x 2048 22.7 -> 25.5, residual 956 x 4096 x 2048 23.9
// -> 24.5, SwiGLU 148 x 16384 x 2048 22.5 -> 23.9; 224 tiles, 788 x 4096 x 2048 of heads 22.1 -> 21.6, residual 21.9 -> 21.4).  Four contexts that call at once share units no worse: six short
// candidates, eight layers of the 0.6B shape 205 us a call with these rings, 206 without.
static constexpr int kNever = 1 << 30;
struct DeepRing {
  int slices, last_rows, full_slices;      // K from `slices` on where the last row tile has up to last_rows rows, else from full_slices on
  int chip_slices;                         // more than 224 tiles: from here on
};
static bool deep_ring(const TileCost &t, bool glu, const DeepRing &r, int64_t M, int64_t ncols, int K) {
  const int bn = glu ? t.bn / 2 : t.bn;
  const int64_t tiles = (M + t.bm - 1) / t.bm * ((ncols + bn - 1) / bn), last = (M - 1) % t.bm + 1;
  return tiles <= 256 && K / BK >= (last <= r.last_rows ? r.slices : r.full_slices) && (tiles <= 224 || K / BK >= r.chip_slices);
}
static bool deep_tile(int kind, int epi, int M, int ncols, int K) {
  const bool glu = epi == PRISM_EPI_SWIGLU;
  if (kind == kTile128Deep) return deep_ring(kTileCost[kind], glu, DeepRing{32, 64, kNever, 48}, M, ncols, K);
  if (kind == kTile128x64)
    return deep_ring(kTileCost[kind], glu, glu ? DeepRing{16, 96, 32, 0} : epi == PRISM_EPI_RESIDUAL ? DeepRing{32, 128, 32, 0} : DeepRing{16, 128, 16, 0}, M, ncols, K);
  return false;
}
static bool deep_head(int kind, int M, int ncols, int K) {
  if (kind == kHead128Deep) return deep_ring(kHeadCost[kind], false, DeepRing{32, 96, kNever, 48}, M, ncols, K);
  return kind == kHead64 && deep_ring(kHeadCost[kind], false, DeepRing{16, 64, 16, 0}, M, ncols, K);
}

template <typename OT, int EPI>
static int launch_kind(int kind, const OT *A, const OT *W, void *out, int M, int N, int K, hipStream_t s) {
  if (deep_tile(kind, EPI, M, EPI == PRISM_EPI_SWIGLU ? N / 2 : N, K)) {
    if (kind == kTile128Deep) return launch_cfg<OT, 128, 128, 2, 2, EPI, 5>(A, W, out, M, N, K, s);
    return launch_cfg<OT, 128, 64, 4, 1, EPI, 6>(A, W, out, M, N, K, s);
  }
  switch (kind) {
    case kTile256: return launch_cfg<OT, 256, 256, 2, 2, EPI, 2>(A, W, out, M, N, K, s);
    case kTile128: return launch_cfg<OT, 128, 128, 2, 2, EPI, 2>(A, W, out, M, N, K, s);
    case kTile128Deep: return launch_cfg<OT, 128, 128, 2, 2, EPI, 4>(A, W, out, M, N, K, s);
    case kTile128x64: return launch_cfg<OT, 128, 64, 4, 1, EPI, 3>(A, W, out, M, N, K, s);
    case kTile64: return launch_cfg<OT, 64, 64, 2, 2, EPI, 5>(A, W, out, M, N, K, s);
    case kTile32x64: return launch_cfg<OT, 32, 64, 1, 1, EPI, 4>(A, W, out, M, N, K, s);
    default: break;
  }
  if constexpr (EPI != PRISM_EPI_SWIGLU) {
    if (kind == kTile64x32) return launch_cfg<OT, 64, 32, 2, 1, EPI, 7>(A, W, out, M, N, K, s);
    return launch_cfg<OT, 32, 32, 2, 2, EPI, 9>(A, W, out, M, N, K, s);
  }
  return PRISM_EUNSUPPORTED;
}

template <typename OT, int EPI>
static int launch_epi(const OT *A, const OT *W, void *out, int M, int N, int K, hipStream_t s) {
  constexpr bool kGlu = EPI == PRISM_EPI_SWIGLU;
  constexpr size_t out_elem = EPI == PRISM_EPI_RESIDUAL || EPI == PRISM_EPI_STORE_F32 ? 4 : 2;
  const int ncols = kGlu ? N / 2 : N;
  const TilePlan p = plan_tiles(kTileCost, kTileKinds, M, ncols, K, kGlu);
  if (p.rows_big > 0) PRISM_TRY((launch_kind<OT, EPI>(kTile256, A, W, out, p.rows_big, N, K, s)));
  return launch_kind<OT, EPI>(p.kind, A + (size_t)p.rows_big * K, W, reinterpret_cast<char *>(out) + (size_t)p.rows_big * ncols * out_elem,
                              M - p.rows_big, N, K, s);
}

template <typename OT>
static int launch_typed(int epilogue, const OT *A, const OT *W, void *out, int M, int N, int K, hipStream_t s) {
  switch (epilogue) {
    case PRISM_EPI_STORE: return launch_epi<OT, PRISM_EPI_STORE>(A, W, out, M, N, K, s);
    case PRISM_EPI_RESIDUAL: return launch_epi<OT, PRISM_EPI_RESIDUAL>(A, W, out, M, N, K, s);
    case PRISM_EPI_STORE_F32: return launch_epi<OT, PRISM_EPI_STORE_F32>(A, W, out, M, N, K, s);
    default: return launch_epi<OT, PRISM_EPI_SWIGLU>(A, W, out, M, N, K, s);
  }
}

// The kernel addresses its operands with 32-bit byte offsets.  W has to fit that; A (and the output rows with it) is
// cut into row panels that do: rows of a GEMM are independent, so the panels are separate launches.
static int rows_per_launch(int K) {
  const int64_t rows = (((int64_t)1 << 32) - 1) / ((int64_t)K * 2);
  return (int)std::max<int64_t>(256, rows / 256 * 256);
}

int launch_gemm_16(int dtype, int epilogue, const void *A, const void *W, void *out, int M, int N, int K, hipStream_t s) {
  PRISM_REQUIRE(A && W && out && M >= 0 && is16(dtype), PRISM_EINVAL, "gemm: bad arguments");
  PRISM_REQUIRE(gemm_16_supported(epilogue, N, K), PRISM_EUNSUPPORTED,
                "gemm: N = %d, K = %d, epilogue %d not supported (K must be a multiple of %d)", N, K, epilogue, BK);
  PRISM_REQUIRE((int64_t)N * K * 2 < ((int64_t)1 << 32) && (int64_t)256 * K * 2 < ((int64_t)1 << 32), PRISM_EUNSUPPORTED,
                "gemm: a weight operand of %d x %d 16-bit elements exceeds 4 GiB", N, K);
  const int step = rows_per_launch(K);
  const int out_cols = epilogue == PRISM_EPI_SWIGLU ? N / 2 : N;
  const size_t out_elem = epilogue == PRISM_EPI_RESIDUAL || epilogue == PRISM_EPI_STORE_F32 ? 4 : 2;
  for (int m0 = 0; m0 < M; m0 += step) {
    const int rows = std::min(step, M - m0);
    const char *a = reinterpret_cast<const char *>(A) + (size_t)m0 * K * 2;
    char *o = reinterpret_cast<char *>(out) + (size_t)m0 * out_cols * out_elem;
    if (dtype == PRISM_DTYPE_BF16) PRISM_TRY(launch_typed<bf16>(epilogue, (const bf16 *)a, (const bf16 *)W, o, rows, N, K, s));
    else PRISM_TRY(launch_typed<f16>(epilogue, (const f16 *)a, (const f16 *)W, o, rows, N, K, s));
  }
  return PRISM_OK;
}

bool gemm_16_qkv_large(int M, int nq, int nkv) {
  return (nq + 2 * nkv) % 2 == 0 && (int64_t)cdiv(M, 256) * ((nq + 2 * nkv) / 2) >= 256;
}

bool gemm_16_qkv_supported(int nq, int nkv, int hd, int K) {
  return hd == 128 && nq > 0 && nkv > 0 && K > 0 && K % BK == 0;          // one head per wavefront
}

template <typename OT>
static int launch_head(int kind, const QkvEpilogue &e, const OT *A, const OT *W, int M, int N, int K, hipStream_t s) {
  if (deep_head(kind, M, N, K)) {
    if (kind == kHead128Deep) return launch_cfg<OT, 128, 128, 4, 1, kEpiQkv, 5>(A, W, e.QK, M, N, K, s, e);
    return launch_cfg<OT, 64, 128, 4, 1, kEpiQkv, 6>(A, W, e.QK, M, N, K, s, e);
  }
  switch (kind) {
    case kHead256: return launch_cfg<OT, 256, 256, 2, 2, kEpiQkv, 2>(A, W, e.QK, M, N, K, s, e);
    case kHead128: return launch_cfg<OT, 128, 128, 4, 1, kEpiQkv, 2>(A, W, e.QK, M, N, K, s, e);
    case kHead128Deep: return launch_cfg<OT, 128, 128, 4, 1, kEpiQkv, 3>(A, W, e.QK, M, N, K, s, e);
    default: return launch_cfg<OT, 64, 128, 4, 1, kEpiQkv, 3>(A, W, e.QK, M, N, K, s, e);
  }
}

template <typename OT>
static int launch_qkv_typed(const QkvEpilogue &e, const OT *A, const OT *W, int M, int N, int K, hipStream_t s) {
  const int step = rows_per_launch(K);
  // an odd number of heads leaves half a 256-wide tile outside the matrix, and that tile's epilogue has no column guard
  const bool wide = (e.nq + 2 * e.nkv) % 2 == 0;
  auto rows_on = [&](int kind, int m0, int rows) {             // every per-row array moves with the rows
    QkvEpilogue p = e;
    p.pos += m0;
    p.vt_col += m0;
    p.QK = reinterpret_cast<char *>(e.QK) + (size_t)m0 * (e.nq + e.nkv) * 128 * 2;
    return launch_head(kind, p, A + (size_t)m0 * K, W, rows, N, K, s);
  };
  for (int m0 = 0; m0 < M; m0 += step) {
    const int rows = std::min(step, M - m0);
    TilePlan p = plan_tiles(kHeadCost, kHeadKinds, rows, N, K, false);
    if (!wide && (p.rows_big > 0 || p.kind == kHead256)) p = {0, kHead128};
    if (p.rows_big > 0) PRISM_TRY(rows_on(kHead256, m0, p.rows_big));
    PRISM_TRY(rows_on(p.kind, m0 + p.rows_big, rows - p.rows_big));
  }
  return PRISM_OK;
}

int launch_gemm_16_qkv(int dtype, const void *Xn, const void *Wqkv, int M, int K, int hd, const QkvEpilogue &e, hipStream_t s) {
  PRISM_REQUIRE(Xn && Wqkv && M >= 0 && is16(dtype) && e.pos && e.vt_col && e.rope_tab_t && e.rope_stride > 0 && e.QK && e.Vt, PRISM_EINVAL,
                "qkv gemm: bad arguments");
  PRISM_REQUIRE(!e.qk_norm || (e.q_gain && e.k_gain), PRISM_EINVAL, "qkv gemm: gains missing");
  PRISM_REQUIRE(gemm_16_qkv_supported(e.nq, e.nkv, hd, K), PRISM_EUNSUPPORTED, "qkv gemm: shape not supported by the fused epilogue");
  const int N = (e.nq + 2 * e.nkv) * 128;
  PRISM_REQUIRE((int64_t)N * K * 2 < ((int64_t)1 << 32) && (int64_t)256 * K * 2 < ((int64_t)1 << 32), PRISM_EUNSUPPORTED,
                "qkv gemm: the weight operand exceeds 4 GiB");
  // one order of every sum, the finishing kernel's, so this gives the bits of prism_op_gemm + prism_op_qkv_finish at every size
  return dtype == PRISM_DTYPE_BF16 ? launch_qkv_typed(e, (const bf16 *)Xn, (const bf16 *)Wqkv, M, N, K, s)
                                   : launch_qkv_typed(e, (const f16 *)Xn, (const f16 *)Wqkv, M, N, K, s);
}

}  // namespace prism
