// fp32 layer contractions for the fp32 mode (small models, 1e-4 parity runs) on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (157 TFLOP/s published, 150 reached by a large product; the vector pipes reach half of that without
// packed instructions), with every edge bounds-checked, so any M, N, K works.  C = A W^T with A [M,K], W [N,K] row-major, fp32 products and sums throughout.
//
// Workgroup tile BM x BN x BK, 4 wavefronts of TM x TN accumulator tiles of 16 x 16.  The 16-wide instruction rather than
// the 32-wide one: half the cycles per step of K on an accumulator, and these launches are short chains, not full pipes.
// A slice goes memory -> registers -> LDS (rows padded by 16 bytes: the 16 rows an operand read touches then start in
// different banks), the next slice's loads in flight while one is multiplied, one barrier per slice.  A lane reads four
// consecutive k of its row as one 16-byte operand chunk and feeds them to four instructions, so instruction s of a
// 16-deep block sums k = s, 4 + s, 8 + s, 12 + s of it; the order is the same for every tile size.
// Layer of the tiny configuration (hidden 256, ffn 688): q/k/v, down and gate/up projections on 354 rows 44, 132 and 52 us
// on the vector pipes -> 5, 9 and 10 us; on 12859 rows 100, 183 and 195 -> 44, 58-64 and 97-107 (71-94 TFLOP/s; boxes differ).
// What is left there: without loads 95 % of the time, without LDS stores or reads 85 % each, with MFMAs alone 74 %.
#include "common.h"

namespace prism {

template <int BM, int BN, int BK, int WM, int WN, int EPI, bool VEC>
__global__ __launch_bounds__(256) void gemm_fp32_kernel(const float *__restrict__ A, const float *__restrict__ W,
                                                        float *__restrict__ out, int M, int N, int K) {
  constexpr bool kGlu = EPI == PRISM_EPI_SWIGLU;             // B tile: BN / 2 gate rows, then the BN / 2 matching up rows
  constexpr int WMT = BM / WM, WNT = BN / WN, TM = WMT / 16, TN = WNT / 16, LD = BK + 4;
  constexpr int Q = BK / 4, NL = (BM + BN) * Q / 256;        // float4s per row, per thread and slice
  static_assert(WM * WN == 4 && (BM + BN) * Q % 256 == 0 && (!kGlu || TN % 2 == 0), "tile");
  __shared__ __align__(16) float lds[2][(BM + BN) * LD];
  const int F = kGlu ? N / 2 : N;                            // output columns
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * (kGlu ? BN / 2 : BN);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / WN, wn = wave % WN;

  f32x4 st[NL];
  auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int idx = threadIdx.x + j * 256, row = idx / Q, k = k0 + idx % Q * 4;
      const bool a = row < BM;
      const int br = row - BM;
      const int c = kGlu ? n0 + (br % (BN / 2)) : n0 + br;
      const bool ok = a ? m0 + row < M : c < F;
      const float *p = a ? A + (int64_t)(m0 + row) * K + k : W + ((int64_t)c + (kGlu && br >= BN / 2 ? F : 0)) * K + k;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
        if (ok && k < K) v = *reinterpret_cast<const f32x4 *>(p);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) if (ok && k + q < K) v[q] = p[q];
      }
      st[j] = v;
    }
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int idx = threadIdx.x + j * 256;
      *reinterpret_cast<f32x4 *>(&lds[buf][idx / Q * LD + idx % Q * 4]) = st[j];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int r16 = lane & 15, k4 = (lane >> 4) * 4;
  const int nk = (K + BK - 1) / BK;
  load(0);
  store(0);
  if (nk > 1) load(BK);
  __syncthreads();
  for (int t = 0; t < nk; ++t) {
    const float *la = lds[t & 1] + (wm * WMT + r16) * LD + k4, *lb = lds[t & 1] + BM * LD + r16 * LD + k4;
#pragma unroll
    for (int kb = 0; kb < BK; kb += 16) {
      f32x4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const f32x4 *>(la + i * 16 * LD + kb);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        // SwiGLU: accumulator tiles j and j + TN / 2 are a gate tile and the up tile of the same columns
        const int row = kGlu ? (j / (TN / 2)) * (BN / 2) + wn * (WNT / 2) + (j % (TN / 2)) * 16 : wn * WNT + j * 16;
        b[j] = *reinterpret_cast<const f32x4 *>(lb + row * LD + kb);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][s], a[i][s], acc[i][j], 0, 0, 0);
    }
    if (t + 1 < nk) {
      store((t + 1) & 1);                                    // its readers finished slice t - 1 before the last barrier
      if (t + 2 < nk) load((t + 2) * BK);
      __syncthreads();
    }
  }
  // W was the first operand: a lane holds row lane % 16 and four consecutive columns of an accumulator tile
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < (kGlu ? TN / 2 : TN); ++j) {
      const int m = m0 + wm * WMT + i * 16 + r16, n = n0 + (kGlu ? wn * (WNT / 2) : wn * WNT) + j * 16 + k4;
      if (m >= M) continue;
      float *o = out + (int64_t)m * F + n;
      f32x4 v = acc[i][j];
      if (kGlu) {
        const f32x4 u = acc[i][j + (kGlu ? TN / 2 : 0)];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = v[q] / (1.0f + expf(-v[q])) * u[q];
      }
      if (VEC && F % 4 == 0) {
        if (n >= F) continue;
        if (EPI == PRISM_EPI_RESIDUAL) v += *reinterpret_cast<const f32x4 *>(o);
        *reinterpret_cast<f32x4 *>(o) = v;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (n + q < F) o[q] = EPI == PRISM_EPI_RESIDUAL ? o[q] + v[q] : v[q];
      }
    }
}

template <int BM, int BN, int BK, int WM, int WN, int EPI, bool VEC>
static void launch_tile(const float *A, const float *W, float *out, int M, int N, int K, hipStream_t s) {
  const int F = EPI == PRISM_EPI_SWIGLU ? N / 2 : N, cols = EPI == PRISM_EPI_SWIGLU ? BN / 2 : BN;
  gemm_fp32_kernel<BM, BN, BK, WM, WN, EPI, VEC><<<dim3(cdiv(F, cols), cdiv(M, BM)), 256, 0, s>>>(A, W, out, M, N, K);
}

// The tile with the least modelled time: K / 256 x (rounds of one tile per compute unit x round + fill) + call, us; tiles from 32
// to 128 rows and columns.  A large tile reads less LDS per product, a small one leaves less of the last round idle and waits less
// for its slices where a unit holds one or two; 64 rows x 32 columns over four waves of 16 rows was the best small one of the shapes
// tried.  SwiGLU's smallest tile has 64 columns (its waves pair gate and up tiles).  Constants: fit to 404 launches (17 to 20000 rows;
// the fp32 configurations' projections, and 256 to 4096 columns at K up to 4096).  Against the best tile of each the rule loses 0.2 % on
// average and 6 % at worst; against 32 x 32 below 512 tiles of 64 x 64 and those from there on, which stood here once, it gains 2 % on average
// and loses 2 % at worst.  us, that border -> now: gate/up 12859 rows 94 -> 89, 20000 140 -> 135, 1500 18.7 -> 16.7; down 6000 30.5 -> 27.8,
// 8000 38.3 -> 33.2; 16000 x 1536 x 1536 690 -> 639.  A fit to K up to 1024 only, without the first round's extra time, put 354 x 2048 x 2048 and
// 150 x 4096 x 4096 on 64 x 64 tiles: 51 and 101 us instead of 40 and 76.
struct TileTime { int bm, bn; double round, fill, call; };
static constexpr TileTime kFp32Tiles[] = {{32, 32, 1.39, 0.58, 2.73}, {64, 32, 2.57, 1.09, 2.57}, {64, 64, 4.78, 1.38, 2.76},
                                          {128, 64, 8.96, 1.98, 3.56}, {128, 128, 17.80, 1.91, 4.79}};
static constexpr TileTime kFp32SmallGlu = {32, 64, 2.69, 0.64, 2.65};

static int fp32_tile(int epilogue, int M, int N, int K) {
  int best = 0;
  double least = 0;
  for (int i = 0; i < 5; ++i) {
    const TileTime &t = i == 0 && epilogue == PRISM_EPI_SWIGLU ? kFp32SmallGlu : kFp32Tiles[i];
    const int64_t tiles = (int64_t)cdiv(M, t.bm) * cdiv(N, t.bn);
    const double time = ((double)((tiles + 255) / 256) * t.round + t.fill) * K / 256 + t.call;
    if (i == 0 || time < least) { best = i; least = time; }
  }
  return best;
}

template <int EPI, bool VEC>
static void launch_tiles(const float *A, const float *W, float *out, int M, int N, int K, hipStream_t s) {
  switch (fp32_tile(EPI, M, N, K)) {
    case 0: launch_tile<32, EPI == PRISM_EPI_SWIGLU ? 64 : 32, 64, 2, 2, EPI, VEC>(A, W, out, M, N, K, s); break;
    case 1: launch_tile<64, 32, 32, 4, 1, EPI, VEC>(A, W, out, M, N, K, s); break;
    case 2: launch_tile<64, 64, 32, 2, 2, EPI, VEC>(A, W, out, M, N, K, s); break;
    case 3: launch_tile<128, 64, 16, 2, 2, EPI, VEC>(A, W, out, M, N, K, s); break;
    default: launch_tile<128, 128, 16, 2, 2, EPI, VEC>(A, W, out, M, N, K, s);
  }
}

int launch_gemm_fp32(int epilogue, const float *A, const float *W, void *out, int M, int N, int K, hipStream_t s) {
  PRISM_REQUIRE(A && W && out && M >= 0 && N > 0 && K > 0, PRISM_EINVAL, "gemm fp32: bad arguments");
  PRISM_REQUIRE(epilogue != PRISM_EPI_SWIGLU || N % 2 == 0, PRISM_EINVAL, "gemm fp32: SwiGLU needs an even row count");
  PRISM_REQUIRE(epilogue == PRISM_EPI_STORE || epilogue == PRISM_EPI_RESIDUAL || epilogue == PRISM_EPI_SWIGLU, PRISM_EINVAL,
                "gemm: unknown epilogue %d", epilogue);
  if (M == 0) return PRISM_OK;
  float *o = (float *)out;
  // rows that start on 16 bytes move four values at a time
  const bool vec = K % 4 == 0 && ((uintptr_t)A | (uintptr_t)W | (uintptr_t)out) % 16 == 0;
  // grid.y is limited to 65535 blocks: very tall operands in panels (rows are independent)
  const int panel = 65535 * 32, F = epilogue == PRISM_EPI_SWIGLU ? N / 2 : N;
  for (int m0 = 0; m0 < M; m0 += panel) {
    const int rows = M - m0 < panel ? M - m0 : panel;
    const float *a = A + (int64_t)m0 * K;
    float *c = o + (int64_t)m0 * F;
    switch (epilogue * 2 + (vec ? 1 : 0)) {
      case PRISM_EPI_STORE * 2 + 1: launch_tiles<PRISM_EPI_STORE, true>(a, W, c, rows, N, K, s); break;
      case PRISM_EPI_STORE * 2: launch_tiles<PRISM_EPI_STORE, false>(a, W, c, rows, N, K, s); break;
      case PRISM_EPI_RESIDUAL * 2 + 1: launch_tiles<PRISM_EPI_RESIDUAL, true>(a, W, c, rows, N, K, s); break;
      case PRISM_EPI_RESIDUAL * 2: launch_tiles<PRISM_EPI_RESIDUAL, false>(a, W, c, rows, N, K, s); break;
      case PRISM_EPI_SWIGLU * 2 + 1: launch_tiles<PRISM_EPI_SWIGLU, true>(a, W, c, rows, N, K, s); break;
      default: launch_tiles<PRISM_EPI_SWIGLU, false>(a, W, c, rows, N, K, s); break;
    }
    PRISM_HIP(hipGetLastError());
  }
  return PRISM_OK;
}

}  // namespace prism
