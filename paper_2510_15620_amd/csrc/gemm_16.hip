// 16-bit-operand layer contractions on the gfx950 matrix cores (paper Sec. 2.2: the reranker's latency is
// dominated by the matrix multiplications of its transformer blocks).
//
// C = A W^T, A [M,K] and W [N,K] row-major, both bf16 or both IEEE half (K-contiguous, which is what
// the MFMA operand registers want: 8 consecutive k per lane), fp32 accumulation in
// v_mfma_f32_16x16x32_{bf16,f16} (256 x 256 tile) or v_mfma_f32_32x32x16_{bf16,f16} (the others): same dense rate, and
// the same bits for the same k in the same order.
//
// Workgroup tile BM x BN x 64, WM x WN wavefronts, each owning a (BM/WM) x (BN/WN) block of the accumulator.  The
// large-launch shape is 256 x 256 with 2 x 2 wavefronts (one per SIMD, 128 x 128 each,
// 256 accumulator registers in AGPRs); launches with few tiles per compute unit take one of seven smaller tiles
// down to 32 x 32 (see the choice at the launcher).  A and W tiles are staged in LDS (a ring of S stages, 256 x 256: three
// of A and two of W; 16-byte chunks XOR-swizzled by row so that the 16- and 32-row operand reads spread over the banks) by direct
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

// silu(g) * u in fp32, rounded to 16 bits by its callers.  The reciprocal instruction (1 ulp) instead of the ten instructions of a
// correctly rounded division, which were half of the SwiGLU epilogue: 13.8 -> 9.2 thousand cycles of a 256 x 256 tile.
__device__ __forceinline__ float silu_mul(float g, float u) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u; }

// LDS bytes of a tile's operand stages
template <int BM, int BN, int S> constexpr int stage_bytes() { return ((BM == 256 ? 3 : S) * BM + S * BN) * BK * 2; }

template <typename OT, int BM, int BN, int WM, int WN, int EPI, int S>
__global__ __launch_bounds__(WM *WN * 64, BM == 256 ? 1 : 2) void gemm_16_kernel(const OT *__restrict__ A,
                                                               const OT *__restrict__ W, void *__restrict__ out_,
                                                               int M, int N, int K, int nM, int nN, QkvEpilogue qe) {
  constexpr int NW = WM * WN;
  constexpr bool kHeads = EPI == kEpiQkv;
  constexpr int WMT = BM / WM, WNT = BN / WN;      // wave tile
  constexpr int TM = WMT / 32, TN = WNT / 32;      // 32x32 accumulator tiles per wave
  // one direct-to-LDS instruction of a wave moves 64 x 16 B = 8 tile rows
  constexpr int A_ITERS = BM / 8 / NW, B_ITERS = BN / 8 / NW;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile/waves mismatch");
  static_assert(EPI != PRISM_EPI_SWIGLU || TN % 2 == 0, "SwiGLU pairs gate and up tiles");
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
  // byte offsets from A / W (both operands are below 4 GiB: checked by the launcher)
  uint32_t gA[A_ITERS], gB[B_ITERS];
#pragma unroll
  for (int j = 0; j < A_ITERS; ++j) {
    const int row = (wave * A_ITERS + j) * 8 + lrow;
    int gr = m0 + row;
    gr = gr < M ? gr : M - 1;
    gA[j] = ((uint32_t)gr * (uint32_t)K + swz(row, lane & 7) * 8) * 2u;
  }
#pragma unroll
  for (int j = 0; j < B_ITERS; ++j) {
    const int row = (wave * B_ITERS + j) * 8 + lrow;
    int gr;
    if (EPI == PRISM_EPI_SWIGLU) {
      const int half = row / (BN / 2), rr = row % (BN / 2);
      gr = n0 + rr; gr = gr < F ? gr : F - 1;
      gr += half * F;
    } else {
      gr = n0 + row; gr = gr < N ? gr : N - 1;
    }
    gB[j] = ((uint32_t)gr * (uint32_t)K + swz(row, lane & 7) * 8) * 2u;
  }
  // ---- LDS rows this lane reads as MFMA operands: row (A) and first column (B) of its first fragment ----
  constexpr bool k16 = BM == 256;                            // 16x16x32 MFMAs: a lane feeds 8 of the 32 k of one of 16 rows,
  const int frow = lane & (k16 ? 15 : 31), kpart = lane >> (k16 ? 4 : 5);   // else 8 of the 16 k of one of 32 rows
  const int rA0 = wm * WMT + frow, rB0 = wn * (EPI == PRISM_EPI_SWIGLU ? WNT / 2 : WNT) + frow;

  f32x16 acc[TM][TN];                                        // k16: cleared by the K loop
  if constexpr (!k16) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  }

  const int nk = K / BK;

  // ---- epilogue geometry (see the epilogue): everything it reads or writes goes along the rows, 16 bytes per lane.
  //      Residual epilogue: the old values of a 32-row block are requested one block ahead, the first block's
  //      before the K loop where registers are left (tiles below 256; the big tile spills).  The same for what the q/k/v
  //      epilogue reads by row: a small tile's loop is a few microseconds, and each dependent load behind it about one.
  //      (28 layers of the 0.6B shape on 391 rows, with the same in the RMSNorm: 2749 -> 2687 us.)
  constexpr bool kEarly = BM < 256;
  constexpr bool kF32Out = EPI == PRISM_EPI_RESIDUAL || EPI == PRISM_EPI_STORE_F32;
  constexpr int ES = kF32Out ? 4 : 2;                               // bytes per output element
  constexpr int OUTW = EPI == PRISM_EPI_SWIGLU ? WNT / 2 : WNT;    // output columns of the wave
  constexpr int RB = OUTW * ES, CPR = RB / 16;                      // bytes / 16-byte chunks per staged row
  constexpr int NR = 1024 / RB, NI = 32 / NR;                       // rows per instruction, instructions per 32-row block
  const int f_row = lane / CPR, f_chunk = lane % CPR;               // lane -> (row within an instruction, chunk)
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
        const int r = i * 32 + rr * NR;
        if (whole || r + f_row < rows_left) old[i & 1][rr] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(old_at + f_off));
        old_at += out_step;
      }
    }
  };


  constexpr int RPB = k16 ? 2 : 1;                                  // rows of a 32-row block that a lane holds
  int row_in[kHeads ? TM * RPB : 1];                                // q, k heads: positions; v heads: V^T columns
  auto load_rows = [&]() __attribute__((always_inline)) {
    if constexpr (kHeads) {
      const int32_t *src = ((n0 + wn * WNT) >> 7) < qe.nq + qe.nkv ? qe.pos : qe.vt_col;
#pragma unroll
      for (int i = 0; i < TM * RPB; ++i) {
        const int row = m0 + wm * WMT + i * (32 / RPB) + frow;
        row_in[i] = src[row < M ? row : M - 1];
      }
    }
  };
  if constexpr (kEarly) {
    if constexpr (kHeads) load_rows();
    else if (full_n) load_old(0, std::false_type{});
  }

  // ---- epilogue.  The W fragment was the instruction's first operand, so the 32 x 32 accumulator block (i, j) is
  //      transposed: a lane holds four runs g = 0..3 of 4 consecutive columns, elements e = 4 g + q, of ONE row of A
  //      (32x32x16: row lane % 32, columns 8 g + 4 (lane / 32) + q) or of two (16x16x32: tile (g / 2, g % 2) of the block, row
  //      16 (g / 2) + lane % 16, columns 16 (g % 2) + 4 (lane / 16) + q); m_of and n_of below.
  //      Written straight from that layout, one store instruction touches 32 rows with 16-32 bytes in each, and
  //      the number of cache lines an instruction touches - not the bytes - is what the memory path charges for
  //      (measured: 12-29 us per 256 x 256 tile, a tenth to a fifth of the tile's time).  So every block of 32 rows goes
  //      through LDS, which is free once the K loop is done: lanes write their row's values, then read back 16 bytes
  //      each along the rows, so that an instruction reads or writes whole lines (2-8 complete rows of the wave's
  //      columns).  LDS requests of one wave are served in order, so no barrier is needed between the two phases.
  auto epilogue = [&]() __attribute__((always_inline)) {
  // Accumulator element (i, j, e), fetched from its accumulation register when it is needed: behind the hand-scheduled
  // loop all 256 of them sit in AGPRs, and read as plain values the compiler would copy the whole set into vector
  // registers at once, leaving none for the epilogue's own arithmetic.
  // (The compiler does not look inside these statements, so the wait between a matrix instruction and the first read
  // of its result is spelled out: every accumulator tile passes through an empty statement, which puts all matrix
  // instructions before it, then 32 idle cycles - more than the deepest instruction needs to retire.  All of these are
  // volatile, which keeps them in this order.)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
  asm volatile("s_nop 15\n\ts_nop 15");
  auto AC = [&](int i, int j, int e) __attribute__((always_inline)) {
    float r;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(acc[i][j][e]));
    return r;
  };
  __syncthreads();              // every wave's operand loads have landed and nobody reads operands any more
  auto m_of = [&](int g) __attribute__((always_inline)) { return k16 ? (g >> 1) * 16 + frow : frow; };
  auto n_of = [&](int g) __attribute__((always_inline)) { return k16 ? (g & 1) * 16 + kpart * 4 : g * 8 + kpart * 4; };
  constexpr int SWZ = CPR >= 16 ? 15 : CPR - 1;                     // chunk rotation by row: spreads a column of 16-byte
                                                                    // writes (one per row) over the banks
  static_assert(32 * RB <= stage_bytes<BM, BN, S>() / NW, "staging block must fit the wave's share of LDS");
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
    dst += (int64_t)i * 32 * pitch;
#pragma unroll
    for (int rr = 0; rr < NI; ++rr) {
      const uint4 v = staged(rr);
      if (i * 32 + rr * NR + f_row < rows_left) __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t *>(dst + off));
      dst += NR * pitch;
    }
  };

  if constexpr (kHeads) {
    // The wave's 128 columns are one head.  A row's 128 values sit in 2 (16x16x32: 4) lanes with the same lane % 32 (% 16);
    // the rotate-half partner of column d is d + 64 = the same register of accumulator block j + 2, so the per-head RMSNorm
    // (cross-lane adds), the rotation and the single rounding all happen on the accumulators.  What the memory path
    // charges for is cache lines touched per instruction, so the cos/sin pairs come from the TRANSPOSED table (the 16 or 32
    // tokens of a load are consecutive positions of a sequence almost always: two to four lines per load instead of
    // one or two per lane) and the finished q / k rows go through the staging block like the other epilogues' outputs.
    static_assert(WNT == 128 && TN == 4, "one head per wavefront");
    typedef typename Mfma<OT>::vec4 vec4;
    const int head = (n0 + wn * WNT) >> 7;                 // wave-uniform
    if constexpr (!kEarly) load_rows();                    // all row blocks' at once: one memory latency, not one per block
    if (head < qe.nq + qe.nkv) {
      const OT *gain = reinterpret_cast<const OT *>(head < qe.nq ? qe.q_gain : qe.k_gain);
      constexpr int NG = k16 ? 2 : 4;                      // distinct column groups of a lane in 32 columns
      vec4 ga[2][NG], gb[2][NG];
      if (qe.qk_norm) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            ga[j][g] = *reinterpret_cast<const vec4 *>(gain + j * 32 + n_of(g));
            gb[j][g] = *reinterpret_cast<const vec4 *>(gain + j * 32 + n_of(g) + 64);
          }
      }
      const int64_t pitch = (int64_t)(qe.nq + qe.nkv) * 128 * 2;
      unsigned char *const qk_w = reinterpret_cast<unsigned char *>(qe.QK) + (int64_t)(m0 + wm * WMT) * pitch + (int64_t)head * 128 * 2;
      const unsigned qk_off = (unsigned)f_row * (unsigned)pitch + (unsigned)f_chunk * 16u;
      // (cos, sin) of (pos, d) sits at [d * stride + pos]: a wave-uniform base per column plus one 32-bit lane offset (in bytes, or
      // the compiler cannot rule out a carry and adds 64-bit addresses per lane).
      // The 32 pairs of block i + 1 are requested before block i is worked on, so the tile pays the memory latency once,
      // not once per block.
      unsigned lane_off[TM * RPB];
#pragma unroll
      for (int i = 0; i < TM * RPB; ++i) lane_off[i] = ((unsigned)(kpart * 4) * (unsigned)qe.rope_stride + (unsigned)row_in[i]) * 8u;
      float2 cs[2][2][4][4];
      auto load_cs = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int d = j * 32 + (k16 ? (g & 1) * 16 : g * 8) + q;         // without the lane's part
              const char *col = reinterpret_cast<const char *>(qe.rope_tab_t + (int64_t)d * qe.rope_stride);
              cs[i & 1][j][g][q] = *reinterpret_cast<const float2 *>(col + lane_off[k16 ? i * 2 + (g >> 1) : i]);
            }
      };
      load_cs(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) load_cs(i + 1);
        float r[RPB];
#pragma unroll
        for (int h = 0; h < RPB; ++h) r[h] = 1.f;
        if (qe.qk_norm) {
          // the finishing kernel's order of the sum of squares: column pairs (d, d + 64), then halving over the bits of d, 32 first
#pragma unroll
          for (int h = 0; h < RPB; ++h) {
            float p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              auto pair = [&](int j, int g) __attribute__((always_inline)) {
                const float a = AC(i, j, g * 4 + q), b = AC(i, j + 2, g * 4 + q);
                return __builtin_fmaf(a, a, b * b);
              };
              auto both = [&](int g) __attribute__((always_inline)) { return pair(0, g) + pair(1, g); };
              if constexpr (k16) p[q] = sum_xor16(sum_xor32(both(h * 2) + both(h * 2 + 1)));
              else p[q] = sum_xor32((both(0) + both(2)) + (both(1) + both(3)));
            }
            r[h] = 1.0f / sqrtf(((p[0] + p[2]) + (p[1] + p[3])) / 128.f + qe.eps);
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            vec4 lo, hi;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float2 c = cs[i & 1][j][g][q];
              float a = AC(i, j, g * 4 + q), b = AC(i, j + 2, g * 4 + q);
              if (qe.qk_norm) {
                a = a * r[k16 ? g >> 1 : 0] * to_f32(ga[j][g % NG][q]);
                b = b * r[k16 ? g >> 1 : 0] * to_f32(gb[j][g % NG][q]);
              }
              lo[q] = from_f32<OT>(__builtin_fmaf(a, c.x, -(b * c.y)));
              hi[q] = from_f32<OT>(__builtin_fmaf(b, c.x, a * c.y));
            }
            put16(m_of(g), j * 32 + n_of(g), lo);
            put16(m_of(g), j * 32 + n_of(g) + 64, hi);
          }
        }
        flush_store(qk_w, pitch, qk_off, i);
      }
    } else {
      // v head: rounded to the operand type, stored as half, transposed (16 or 32 consecutive tokens of one d are contiguous)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int h = 0; h < RPB; ++h) {
          if (m0 + wm * WMT + i * 32 + h * 16 + frow >= M) continue;
          f16 *vt = reinterpret_cast<f16 *>(qe.Vt) + ((int64_t)(head - qe.nq - qe.nkv) * 128 + kpart * 4) * qe.vt_stride + row_in[i * RPB + h];
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int g = h * 2; g < h * 2 + 4 / RPB; ++g)
#pragma unroll
              for (int q = 0; q < 4; ++q)
                vt[(int64_t)(j * 32 + (k16 ? (g & 1) * 16 : g * 8) + q) * qe.vt_stride] = from_f32<f16>(to_f32(from_f32<OT>(AC(i, j, g * 4 + q))));
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
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) load_old(i + 1, whole);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = AC(i, j, g * 4 + q);
            put32(m_of(g), j * 32 + n_of(g), v);
          }
#pragma unroll
        for (int rr = 0; rr < NI; ++rr) {
          const int r = i * 32 + rr * NR;
          const uint4 u = staged(rr);
          f32x4 v = old[i & 1][rr];
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
    for (int i = 0; i < TM; ++i) {
      if (EPI == PRISM_EPI_SWIGLU) {
#pragma unroll
        for (int j = 0; j < TN / 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            typename Mfma<OT>::vec4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = from_f32<OT>(silu_mul(AC(i, j, g * 4 + q), AC(i, j + TN / 2, g * 4 + q)));
            put16(m_of(g), j * 32 + n_of(g), v);
          }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            if (EPI == PRISM_EPI_STORE_F32) {
              f32x4 v;
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = AC(i, j, g * 4 + q);
              put32(m_of(g), j * 32 + n_of(g), v);
            } else {
              typename Mfma<OT>::vec4 v;
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = from_f32<OT>(AC(i, j, g * 4 + q));
              put16(m_of(g), j * 32 + n_of(g), v);
            }
          }
      }
      flush_store(out_w, out_pitch, f_off, i);
    }
    return;
  }

  // ---- ragged last column tile (N not a multiple of the tile, or rows not 16-byte aligned): element by element
  if constexpr (!kHeads) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < (EPI == PRISM_EPI_SWIGLU ? TN / 2 : TN); ++j)
        for (int g = 0; g < 4; ++g)
          for (int q = 0; q < 4; ++q) {
            const int row = m0 + wm * WMT + i * 32 + m_of(g), col = n0 + wn * OUTW + j * 32 + n_of(g) + q;
            if (row >= M || col >= F) continue;
            if (EPI == PRISM_EPI_SWIGLU) {
              reinterpret_cast<OT *>(out_)[(int64_t)row * F + col] = from_f32<OT>(silu_mul(AC(i, j, g * 4 + q), AC(i, j + TN / 2, g * 4 + q)));
            } else if (EPI == PRISM_EPI_RESIDUAL) {
              reinterpret_cast<float *>(out_)[(int64_t)row * N + col] += AC(i, j, g * 4 + q);
            } else if (EPI == PRISM_EPI_STORE_F32) {
              reinterpret_cast<float *>(out_)[(int64_t)row * N + col] = AC(i, j, g * 4 + q);
            } else {
              reinterpret_cast<OT *>(out_)[(int64_t)row * N + col] = from_f32<OT>(AC(i, j, g * 4 + q));
            }
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
  const uint64_t baseA = (uint64_t)(uintptr_t)A, baseB = (uint64_t)(uintptr_t)W;
  constexpr bool kF16 = Mfma<OT>::kIsF16;
  if constexpr (BM < 256) {
#define PRISM_ACC1 "+a"(acc[0][0])
#define PRISM_ACC2 PRISM_ACC1, "+a"(acc[0][1])
#define PRISM_ACC4 PRISM_ACC2, "+a"(acc[1][0]), "+a"(acc[1][1])
#define PRISM_ACC1x4 PRISM_ACC2, "+a"(acc[0][2]), "+a"(acc[0][3])
#define PRISM_G2(g) "v"(g[0]), "v"(g[1])
#define PRISM_G4(g) PRISM_G2(g), "v"(g[2]), "v"(g[3])
#define PRISM_G8(g) PRISM_G4(g), "v"(g[4]), "v"(g[5]), "v"(g[6]), "v"(g[7])
#define PRISM_RUN_SMALL(NAME, ACC, GA, GB)                                                                              \
  do {                                                                                                                  \
    if constexpr (kF16)                                                                                                 \
      asm volatile(PRISM_KLOOP_F16_##NAME : ACC : "v"(aA0), "v"(aB0), GA(gA), GB(gB), "s"(ldsA_w), "s"(ldsB_w),         \
                   "s"(baseA), "s"(baseB), "s"(nk) : PRISM_KLOOP_CLOBBERS_##NAME);                                      \
    else                                                                                                                \
      asm volatile(PRISM_KLOOP_BF16_##NAME : ACC : "v"(aA0), "v"(aB0), GA(gA), GB(gB), "s"(ldsA_w), "s"(ldsB_w),        \
                   "s"(baseA), "s"(baseB), "s"(nk) : PRISM_KLOOP_CLOBBERS_##NAME);                                      \
  } while (0)
    if constexpr (kHeads) {
      if constexpr (BM == 64) PRISM_RUN_SMALL(64x128_3_HEAD, PRISM_ACC1x4, PRISM_G4, PRISM_G8);
      else if constexpr (S == 3) PRISM_RUN_SMALL(128x128_3_HEAD, PRISM_ACC1x4, PRISM_G4, PRISM_G4);
      else PRISM_RUN_SMALL(128x128_2_HEAD, PRISM_ACC1x4, PRISM_G4, PRISM_G4);
    } else if constexpr (BM == 32 && BN == 32) PRISM_RUN_SMALL(32x32_8, PRISM_ACC1, PRISM_G4, PRISM_G4);
    else if constexpr (BM == 64 && BN == 32) PRISM_RUN_SMALL(64x32_6, PRISM_ACC1, PRISM_G4, PRISM_G2);
    else if constexpr (BM == 32 && BN == 64) PRISM_RUN_SMALL(32x64_4, PRISM_ACC2, PRISM_G4, PRISM_G8);
    else if constexpr (BM == 64 && BN == 64) PRISM_RUN_SMALL(64x64_5, PRISM_ACC2, PRISM_G4, PRISM_G4);
    else if constexpr (BM == 128 && BN == 64) PRISM_RUN_SMALL(128x64_3, PRISM_ACC2, PRISM_G4, PRISM_G2);
    else if constexpr (S == 3 && EPI == PRISM_EPI_SWIGLU) PRISM_RUN_SMALL(128x128_3_SWIGLU, PRISM_ACC4, PRISM_G4, PRISM_G4);
    else if constexpr (S == 3) PRISM_RUN_SMALL(128x128_3_PLAIN, PRISM_ACC4, PRISM_G4, PRISM_G4);
    else if constexpr (EPI == PRISM_EPI_SWIGLU) PRISM_RUN_SMALL(128x128_2_SWIGLU, PRISM_ACC4, PRISM_G4, PRISM_G4);
    else PRISM_RUN_SMALL(128x128_2_PLAIN, PRISM_ACC4, PRISM_G4, PRISM_G4);
  } else {
    // the second 64 columns of the wave: SwiGLU's are the up rows, half a tile further (the swizzle repeats every 16 rows)
    const unsigned aB1 = aB0 + (unsigned)((EPI == PRISM_EPI_SWIGLU ? BN / 2 : 64) * BK) * 2u;
#define PRISM_AB(j) [ga##j] "v"(gA[j]), [gb##j] "v"(gB[j])
#define PRISM_RUN_KLOOP(TY)                                                                                                    \
  asm volatile(PRISM_KLOOP_256(TY)                                                                                             \
               : "={a[0:15]}"(acc[0][0]), "={a[16:31]}"(acc[0][1]), "={a[32:47]}"(acc[0][2]), "={a[48:63]}"(acc[0][3]),          \
                 "={a[64:79]}"(acc[1][0]), "={a[80:95]}"(acc[1][1]), "={a[96:111]}"(acc[1][2]), "={a[112:127]}"(acc[1][3]),      \
                 "={a[128:143]}"(acc[2][0]), "={a[144:159]}"(acc[2][1]), "={a[160:175]}"(acc[2][2]), "={a[176:191]}"(acc[2][3]), \
                 "={a[192:207]}"(acc[3][0]), "={a[208:223]}"(acc[3][1]), "={a[224:239]}"(acc[3][2]), "={a[240:255]}"(acc[3][3])  \
               : [aa] "v"(aA0), [ab] "v"(aB0), [ab2] "v"(aB1), PRISM_AB(0), PRISM_AB(1), PRISM_AB(2), PRISM_AB(3), PRISM_AB(4),  \
                 PRISM_AB(5), PRISM_AB(6), PRISM_AB(7), [la] "s"(ldsA_w), [lb] "s"(ldsB_w), [pa] "s"(baseA), [pb] "s"(baseB),     \
                 [nk] "s"(nk)                                                                                                   \
               : PRISM_KLOOP_256_CLOBBERS)
    if constexpr (kF16) PRISM_RUN_KLOOP("f16");
    else PRISM_RUN_KLOOP("bf16");
#undef PRISM_RUN_KLOOP
  }
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
// many tiles share the unit: alone it is a chain of latencies, together the matrix pipes and LDS.  The constants describe
// every tile size on 171 launches (N 1024-24576, K 1024-12288, 1 to 20000 rows, three epilogues) within 12-18 % (root mean
// square); the size picked by them is on average within 1 % of the best one measured, at worst 9 %.  Examples, in us, 128 x 128
// compiler-scheduled loop before -> now: 100 x 4096 x 12288 167 -> 36 (64 x 32), 391 x 1024 x 3072 44 -> 10 (64 x 32),
// 777 x 6144 x 1024 with SwiGLU 23 -> 17 (128 x 128), 3699 x 1024 x 3072 49 -> 30 (128 x 128, three stages).
// (256 x 256: on chips of different speed a slice takes 1.34-1.7 us, the fixed part 11 us with SwiGLU and 17 with a residual or a
// head; 1024 x 24576 x 4096 with SwiGLU 233 us on 128 x 128 tiles, 203 on these; 1536 x 6144 x 4096 with heads 103 and 90.)
struct TileCost {
  int bm, bn, occ;              // tile, workgroups that share a compute unit
  float alone, shared, fixed;   // us per 64-deep slice: one workgroup on the unit; per workgroup when occ of them share it; us per tile
};
enum { kTile256, kTile128, kTile128Deep, kTile128x64, kTile64, kTile32x64, kTile64x32, kTile32, kTileKinds };
static constexpr TileCost kTileCost[kTileKinds] = {
    {256, 256, 1, 1.45f, 1.45f, 9.2f}, {128, 128, 2, 0.72f, 0.50f, 4.5f}, {128, 128, 1, 0.52f, 0.52f, 3.4f}, {128, 64, 2, 0.34f, 0.36f, 2.3f},
    {64, 64, 2, 0.204f, 0.204f, 2.1f}, {32, 64, 3, 0.176f, 0.149f, 2.4f}, {64, 32, 2, 0.128f, 0.128f, 2.3f}, {32, 32, 2, 0.106f, 0.083f, 2.6f}};
// The fused q/k/v projection: tiles whose waves own whole heads (34 launches of 1 to 12000 rows: within 11-19 %, the picked
// size on average within 1 % of the best, at worst 12 %).  Its epilogue is longer: two dependent loads (position, rotation)
// and the per-head arithmetic.  391 x 4096 x 1024: 11 us, where the projection to fp32 and its two finishing kernels took 48;
// 777 x 6144 x 4096: 56.
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

template <typename OT, int EPI>
static int launch_kind(int kind, const OT *A, const OT *W, void *out, int M, int N, int K, hipStream_t s) {
  switch (kind) {
    case kTile256: return launch_cfg<OT, 256, 256, 2, 2, EPI, 2>(A, W, out, M, N, K, s);
    case kTile128: return launch_cfg<OT, 128, 128, 2, 2, EPI, 2>(A, W, out, M, N, K, s);
    case kTile128Deep: return launch_cfg<OT, 128, 128, 2, 2, EPI, 3>(A, W, out, M, N, K, s);
    case kTile128x64: return launch_cfg<OT, 128, 64, 4, 1, EPI, 3>(A, W, out, M, N, K, s);
    case kTile64: return launch_cfg<OT, 64, 64, 2, 1, EPI, 5>(A, W, out, M, N, K, s);
    case kTile32x64: return launch_cfg<OT, 32, 64, 1, 1, EPI, 4>(A, W, out, M, N, K, s);
    default: break;
  }
  if constexpr (EPI != PRISM_EPI_SWIGLU) {
    if (kind == kTile64x32) return launch_cfg<OT, 64, 32, 2, 1, EPI, 6>(A, W, out, M, N, K, s);
    return launch_cfg<OT, 32, 32, 1, 1, EPI, 8>(A, W, out, M, N, K, s);
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
  switch (kind) {
    case kHead256: return launch_cfg<OT, 256, 256, 2, 2, kEpiQkv, 2>(A, W, e.QK, M, N, K, s, e);
    case kHead128: return launch_cfg<OT, 128, 128, 4, 1, kEpiQkv, 2>(A, W, e.QK, M, N, K, s, e);
    case kHead128Deep: return launch_cfg<OT, 128, 128, 4, 1, kEpiQkv, 3>(A, W, e.QK, M, N, K, s, e);
    default: return launch_cfg<OT, 64, 128, 2, 1, kEpiQkv, 3>(A, W, e.QK, M, N, K, s, e);
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
