// Bandwidth- and latency-bound steps of the path: embedding gather, RMSNorm, q/k norm + RoPE,
// V rounding + transposition, the intermediate scorer, compaction and the final top-K.
#include <type_traits>

#include "common.h"

namespace prism {

// ------------------------------------------------------------------------------------------------
// Pack + embed: X[t,:] = table[tokens[t],:]            (paper Sec. 4.5: forwarding begins at the embedding)
// One workgroup per token row; HBM-bound (T*H*4 B written).
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const int32_t *__restrict__ tokens, const T *__restrict__ table,
                                                    int hidden, float *__restrict__ X) {
  const int64_t t = blockIdx.x;
  const T *src = table + (int64_t)tokens[t] * hidden;
  float *dst = X + t * hidden;
  for (int i = threadIdx.x * 4; i < hidden; i += blockDim.x * 4) {
    if (i + 3 < hidden) {
      float4 v = make_float4(to_f32(src[i]), to_f32(src[i + 1]), to_f32(src[i + 2]), to_f32(src[i + 3]));
      *reinterpret_cast<float4 *>(dst + i) = v;
    } else {
      for (int j = i; j < hidden; ++j) dst[j] = to_f32(src[j]);
    }
  }
}

int launch_embed(const int32_t *tokens, int T, const void *table, int hidden, int dtype, float *X, hipStream_t s) {
  PRISM_REQUIRE(tokens && table && X && T >= 0 && hidden > 0 && hidden % 4 == 0, PRISM_EINVAL, "embed: bad arguments");
  if (T == 0) return PRISM_OK;
  if (dtype == PRISM_DTYPE_FP32)
    embed_kernel<float><<<T, 256, 0, s>>>(tokens, (const float *)table, hidden, X);
  else
    embed_kernel<bf16><<<T, 256, 0, s>>>(tokens, (const bf16 *)table, hidden, X);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// RMSNorm of the fp32 residual into the GEMM operand type.  One workgroup per row.  HBM-bound: T*H*(4 + sizeof(T)) bytes.
__device__ __forceinline__ float block_sum_256(float v, float *red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float t = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return t;
}

template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float *__restrict__ X, const T *__restrict__ gain,
                                                      int hidden, float eps, T *__restrict__ out) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  __shared__ float red[4];
  const float *x = X + (int64_t)blockIdx.x * hidden;
  T *o = out + (int64_t)blockIdx.x * hidden;
  // NV > 0: the row (at most NV * 1024 values) stays in registers between the two passes; it is not needed again before
  // the layer's next GEMM epilogue, so the loads bypass the caches' retention.  NV == 0: any width, the row is read twice.
  // The gains are requested with the row, not behind the sum: a launch of a few hundred rows is one round of latencies.
  struct alignas(sizeof(T) * 4) Quad { T v[4]; } g[NV > 0 ? NV : 1];
  f32x4_t keep[NV > 0 ? NV : 1];
  float ss = 0.f;
  if (NV > 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = threadIdx.x * 4 + k * 1024;
      if (i < hidden) {
        keep[k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(x + i));
        g[k] = *reinterpret_cast<const Quad *>(gain + i);
        ss += keep[k][0] * keep[k][0] + keep[k][1] * keep[k][1] + keep[k][2] * keep[k][2] + keep[k][3] * keep[k][3];
      }
    }
  } else {
    for (int i = threadIdx.x * 4; i < hidden; i += 1024) {
      float4 v = *reinterpret_cast<const float4 *>(x + i);
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
  }
  ss = block_sum_256(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
  auto emit = [&](int i, float a, float b, float c, float d, const Quad &g) {
    Quad q;
    q.v[0] = from_f32<T>(a * r * to_f32(g.v[0]));
    q.v[1] = from_f32<T>(b * r * to_f32(g.v[1]));
    q.v[2] = from_f32<T>(c * r * to_f32(g.v[2]));
    q.v[3] = from_f32<T>(d * r * to_f32(g.v[3]));
    *reinterpret_cast<Quad *>(o + i) = q;
  };
  if (NV > 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = threadIdx.x * 4 + k * 1024;
      if (i < hidden) emit(i, keep[k][0], keep[k][1], keep[k][2], keep[k][3], g[k]);
    }
  } else {
    for (int i = threadIdx.x * 4; i < hidden; i += 1024) {
      float4 v = *reinterpret_cast<const float4 *>(x + i);
      emit(i, v.x, v.y, v.z, v.w, *reinterpret_cast<const Quad *>(gain + i));
    }
  }
}

// Rows of up to 256 values: one wave each.  In the kernel above three of a row's four waves would idle; the sum is that
// of the first, in its order, so the bits are the same.  12859 rows of 256: 11-12 -> 5.6-6.8 us.  (Rows of 1024 in one wave, four
// sums side by side, took 5.5 us instead of 4.2 on 391 rows and 8.2 instead of 7.2 on 3700-12100: they stay with a workgroup.)
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_short_kernel(const float *__restrict__ X, const T *__restrict__ gain, int n_rows, int hidden,
                                                            float eps, T *__restrict__ out) {
  const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), i = (threadIdx.x & 63) * 4;
  if (row >= n_rows) return;
  struct alignas(sizeof(T) * 4) Quad { T v[4]; } g, q;
  f32x4 keep;
  float ss = 0.f;
  if (i < hidden) {
    keep = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(X + (int64_t)row * hidden + i));
    g = *reinterpret_cast<const Quad *>(gain + i);
    ss += keep[0] * keep[0] + keep[1] * keep[1] + keep[2] * keep[2] + keep[3] * keep[3];
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
  if (i >= hidden) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) q.v[e] = from_f32<T>(keep[e] * r * to_f32(g.v[e]));
  *reinterpret_cast<Quad *>(out + (int64_t)row * hidden + i) = q;
}

template <typename T>
static void launch_rmsnorm_typed(const float *X, const void *gain, int T_, int hidden, float eps, void *out, hipStream_t s) {
  const int rows = T_ >= 4096 ? 4 : 1;                       // of a workgroup: a few hundred rows reach every compute unit one by one
  if (hidden <= 256) rmsnorm_short_kernel<T><<<cdiv(T_, rows), rows * 64, 0, s>>>(X, (const T *)gain, T_, hidden, eps, (T *)out);
  else if (hidden <= 4096) rmsnorm_kernel<T, 4><<<T_, 256, 0, s>>>(X, (const T *)gain, hidden, eps, (T *)out);
  else if (hidden <= 8192) rmsnorm_kernel<T, 8><<<T_, 256, 0, s>>>(X, (const T *)gain, hidden, eps, (T *)out);
  else rmsnorm_kernel<T, 0><<<T_, 256, 0, s>>>(X, (const T *)gain, hidden, eps, (T *)out);
}

int launch_rmsnorm(const float *X, const void *gain, int T, int hidden, float eps, int dtype, void *out, hipStream_t s) {
  PRISM_REQUIRE(X && gain && out && T >= 0 && hidden > 0 && hidden % 4 == 0, PRISM_EINVAL, "rmsnorm: bad arguments");
  const size_t quad = 4 * dtype_size(dtype);        // the kernel moves four values at a time
  PRISM_REQUIRE((uintptr_t)X % 16 == 0 && (uintptr_t)gain % quad == 0 && (uintptr_t)out % quad == 0, PRISM_EINVAL,
                "rmsnorm: X must be 16-byte aligned, gain and out %zu-byte aligned", quad);
  if (T == 0) return PRISM_OK;
  if (dtype == PRISM_DTYPE_FP32) launch_rmsnorm_typed<float>(X, gain, T, hidden, eps, out, s);
  else if (dtype == PRISM_DTYPE_BF16) launch_rmsnorm_typed<bf16>(X, gain, T, hidden, eps, out, s);
  else launch_rmsnorm_typed<f16>(X, gain, T, hidden, eps, out, s);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// RoPE table, evaluated in fp64 and rounded once: (cos, sin)(pos * base^(-2 i / hd)) at tab[pos * half + i], or, transposed,
// at tab[i * n_pos + pos] (the layout the fused q/k/v epilogue reads: consecutive tokens of a sequence are then neighbours).
__device__ __forceinline__ float2 rotation(int pos, int i, int half, double log2_base) {
  const double theta = exp2(-(double)i / (double)half * log2_base);
  const double a = (double)pos * theta;
  return make_float2((float)cos(a), (float)sin(a));
}

__global__ void rope_table_kernel(float2 *tab, int n_pos, int half, double log2_base, int transposed) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_pos * half) return;
  const int pos = transposed ? idx % n_pos : idx / half, i = transposed ? idx / n_pos : idx % half;
  tab[idx] = rotation(pos, i, half, log2_base);
}

int launch_rope_table(float2 *tab, int n_pos, int head_dim, float rope_base, hipStream_t s, bool transposed) {
  PRISM_REQUIRE(tab && n_pos > 0 && head_dim > 0 && head_dim % 2 == 0 && rope_base > 0, PRISM_EINVAL, "rope table: bad arguments");
  const int half = head_dim / 2, n = n_pos * half;
  rope_table_kernel<<<cdiv(n, 256), 256, 0, s>>>(tab, n_pos, half, log2((double)rope_base), transposed ? 1 : 0);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// Row copy between two tables by index lists: one workgroup per row, 16 bytes per lane and step.
__global__ __launch_bounds__(256) void copy_rows_kernel(const uint4 *__restrict__ src, const int32_t *__restrict__ src_idx,
                                                        uint4 *__restrict__ dst, const int32_t *__restrict__ dst_idx, int vecs) {
  const uint4 *a = src + (int64_t)src_idx[blockIdx.x] * vecs;
  uint4 *b = dst + (int64_t)dst_idx[blockIdx.x] * vecs;
  for (int i = threadIdx.x; i < vecs; i += 256) b[i] = a[i];
}

int launch_copy_rows(const void *src, const int32_t *src_idx, void *dst, const int32_t *dst_idx, int n, size_t row_bytes,
                     hipStream_t s) {
  PRISM_REQUIRE(src && src_idx && dst && dst_idx && n >= 0 && row_bytes % 16 == 0, PRISM_EINVAL, "copy_rows: bad arguments");
  if (n == 0) return PRISM_OK;
  copy_rows_kernel<<<n, 256, 0, s>>>((const uint4 *)src, src_idx, (uint4 *)dst, dst_idx, (int)(row_bytes / 16));
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// The rows a checked or last layer goes on with, out of two tables at once (attention output and residual): row i of dst0 and
// dst1 = row idx[i] of src0 and src1.  Launch-bound (4.6 us each as two copies): one launch, blockIdx.y picks the table.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4 *__restrict__ src0, const uint4 *__restrict__ src1,
                                                          const int32_t *__restrict__ idx, uint4 *__restrict__ dst0,
                                                          uint4 *__restrict__ dst1, int vecs0, int vecs1) {
  const int vecs = blockIdx.y ? vecs1 : vecs0;
  const uint4 *a = (blockIdx.y ? src1 : src0) + (int64_t)idx[blockIdx.x] * vecs;
  uint4 *b = (blockIdx.y ? dst1 : dst0) + (int64_t)blockIdx.x * vecs;
  for (int i = threadIdx.x; i < vecs; i += 256) b[i] = a[i];
}

int launch_gather_rows(const void *src0, const void *src1, const int32_t *idx, void *dst0, void *dst1, int n, size_t row_bytes0,
                       size_t row_bytes1, hipStream_t s) {
  PRISM_REQUIRE(src0 && src1 && idx && dst0 && dst1 && n >= 0 && row_bytes0 % 16 == 0 && row_bytes1 % 16 == 0, PRISM_EINVAL,
                "gather_rows: bad arguments");
  if (n == 0) return PRISM_OK;
  gather_rows_kernel<<<dim3(n, 2), 256, 0, s>>>((const uint4 *)src0, (const uint4 *)src1, idx, (uint4 *)dst0, (uint4 *)dst1,
                                                 (int)(row_bytes0 / 16), (int)(row_bytes1 / 16));
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// Per-head RMSNorm (optional) then rotate-half RoPE on the q and k parts of the fp32 projection
// QKV [T, (nq + 2 nkv) * hd].  One wavefront per (token, head); lane i owns pairs (i, i + hd/2),
// (i + 64, i + 64 + hd/2), ...  The result is rounded ONCE, to the operand type of the QK^T
// contraction: fp32 mode rewrites QKV in place, bf16 mode writes QK [T, (nq + nkv) * hd].
template <typename T>
__global__ __launch_bounds__(256) void qk_finish_kernel(float *__restrict__ QKV, const int32_t *__restrict__ pos,
                                                        const T *__restrict__ q_gain, const T *__restrict__ k_gain,
                                                        int n_tok, int nq, int nkv, int hd, float eps, int qk_norm,
                                                        const float2 *__restrict__ rope_tab, T *__restrict__ out,
                                                        int out_row) {
  const int heads = nq + nkv;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= (int64_t)n_tok * heads) return;
  const int t = (int)(item / heads), h = (int)(item % heads);
  const int lane = threadIdx.x & 63, half = hd / 2;
  const float *x = QKV + (int64_t)t * (nq + 2 * nkv) * hd + (int64_t)h * hd;
  T *o = out + (int64_t)t * out_row + (int64_t)h * hd;
  const T *g = h < nq ? q_gain : k_gain;
  const float2 *tab = rope_tab + (int64_t)pos[t] * half;
  float ss = 0.f;
  for (int i = lane; i < half; i += 64) {
    const float a = x[i], b = x[i + half];
    ss += a * a + b * b;
  }
  float r = 1.f;
  if (qk_norm) {
    ss = wave_sum(ss);
    r = 1.0f / sqrtf(ss / (float)hd + eps);
  }
  for (int i = lane; i < half; i += 64) {
    float a = x[i], b = x[i + half];
    if (qk_norm) {
      a = a * r * to_f32(g[i]);
      b = b * r * to_f32(g[i + half]);
    }
    const float2 cs = tab[i];
    o[i] = from_f32<T>(a * cs.x - b * cs.y);
    o[i + half] = from_f32<T>(b * cs.x + a * cs.y);
  }
}

// The same and the V part in one launch, for the 16-bit modes at head_dim 128.  Launch- and latency-bound at the sizes it is
// for (the fused projection serves large ones).  V first: a workgroup takes 64 tokens of one head through LDS, and they leave
// as 64 consecutive tokens of one d per wave instruction.  Then q and k: a workgroup takes all heads of 4 tokens, 16 lanes each,
// a lane holding 4 + 4 values of the two rotation halves; a lane's token stays the same over its heads.  So the tokens' 4 x 64
// rotations are one fp64 evaluation per thread, while the first values are on their way, and no table has to be allocated,
// filled and waited for: 1154 tokens of 16 + 8 heads 3.0 (table) + 9.9 us in two launches -> 9.8 in one.  More than 4 kHeads heads go in
// rounds whose loads wait for the round before: the call with 32 + 8 heads, 391 tokens 23.9 -> 23.6 us, 12 859 135 -> 106.  kFew, for up to 6 heads of
// many tokens: a wave takes all heads of 4 tokens of its own, 16 to a workgroup.  With 4 to a workgroup most waves have a head or
// none, and starting workgroups is what the launch takes its time for: us of the call, by the two launches, 4 tokens and 16: 1 + 1 heads 96 064
// tokens 72, 83, 60, 20 000 33.5, 31.8, 28.3; 2 + 1 of 200 000 154, 209, 139; 4 + 2 of 50 000 89, 86, 71.  Up to some 8000 tokens the
// evaluations of four rotations in a row are the longer way (400 tokens 18.3, 16 to a workgroup 19.7), and from 8 + 2 heads on it is level or worse.
template <typename T, bool kFew>
__global__ __launch_bounds__(256) void qkv_finish_16_kernel(const float *__restrict__ QKV, const int32_t *__restrict__ pos,
                                                            const T *__restrict__ q_gain, const T *__restrict__ k_gain, int n_tok,
                                                            int nq, int nkv, float eps, int qk_norm, double log2_base, T *__restrict__ out,
                                                            f16 *__restrict__ Vt, const int32_t *__restrict__ vt_col, int64_t vt_stride) {
  constexpr int HD = 128, kTok = kFew ? 16 : 4, kHeads = 6;  // tokens of a workgroup, heads whose values a lane requests together
  constexpr int kStep = kFew ? 1 : 4;                        // from one head of a wave to its next
  typedef typename Mfma<T>::vec4 vec4;
  const int heads = nq + nkv, row = (nq + 2 * nkv) * HD;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int v_groups = (n_tok + 63) / 64 * nkv;
  if ((int)blockIdx.x >= v_groups) {
    __shared__ __align__(16) float2 rot[kTok][HD / 2];
    const int t0 = ((int)blockIdx.x - v_groups) * kTok, h_first = kFew ? 0 : wave;
    const int i = (lane & 15) * 4, tk = (kFew ? wave * 4 : 0) + (lane >> 4);   // first of the lane's 4 rotation pairs, its token
    const int t = t0 + tk < n_tok ? t0 + tk : n_tok - 1;
    int rpos[kTok / 4];                                      // positions of the tokens whose rotations this wave evaluates
#pragma unroll
    for (int r = 0; r < kTok / 4; ++r) {
      const int rt = t0 + wave * (kTok / 4) + r;
      rpos[r] = pos[rt < n_tok ? rt : n_tok - 1];
    }
    vec4 gq[2], gk[2];
    if (qk_norm) {
      gq[0] = *reinterpret_cast<const vec4 *>(q_gain + i);
      gq[1] = *reinterpret_cast<const vec4 *>(q_gain + i + 64);
      gk[0] = *reinterpret_cast<const vec4 *>(k_gain + i);
      gk[1] = *reinterpret_cast<const vec4 *>(k_gain + i + 64);
    }
    const float *x = QKV + (int64_t)t * row + i;
    T *o = out + (int64_t)t * heads * HD + i;
    f32x4 a[kHeads], b[kHeads];
    auto fetch = [&](int h0) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < kHeads; ++k) {
        const int h = h0 + kStep * k < heads ? h0 + kStep * k : heads - 1;
        a[k] = *reinterpret_cast<const f32x4 *>(x + h * HD);
        b[k] = *reinterpret_cast<const f32x4 *>(x + h * HD + 64);
      }
    };
    fetch(h_first);
#pragma unroll
    for (int r = 0; r < kTok / 4; ++r) rot[wave * (kTok / 4) + r][lane] = rotation(rpos[r], lane, HD / 2, log2_base);
    __syncthreads();
    float2 cs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) cs[q] = rot[tk][i + q];
    for (int h0 = h_first; h0 < heads; h0 += kStep * kHeads) {
      if (h0 != h_first) fetch(h0);
#pragma unroll
      for (int k = 0; k < kHeads; ++k) {
        const int h = h0 + kStep * k;
        if (h >= heads) break;                               // the same for the whole wave
        float r = 1.f;
        if (qk_norm) {
          // pairs (d, d + 64), then halving over the bits of d, 32 first: the order of wave_sum with a pair per lane
          float p[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            p[q] = __builtin_fmaf(a[k][q], a[k][q], b[k][q] * b[k][q]);
#pragma unroll
            for (int m = 8; m > 0; m >>= 1) p[q] += __shfl_xor(p[q], m, 64);
          }
          const float ss = (p[0] + p[2]) + (p[1] + p[3]);
          r = 1.0f / sqrtf(ss / (float)HD + eps);
        }
        vec4 lo, hi;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float u = a[k][q], v = b[k][q];
          if (qk_norm) {
            u = u * r * to_f32(h < nq ? gq[0][q] : gk[0][q]);
            v = v * r * to_f32(h < nq ? gq[1][q] : gk[1][q]);
          }
          lo[q] = from_f32<T>(__builtin_fmaf(u, cs[q].x, -(v * cs[q].y)));
          hi[q] = from_f32<T>(__builtin_fmaf(v, cs[q].x, u * cs[q].y));
        }
        if (t0 + tk < n_tok) {
          *reinterpret_cast<vec4 *>(o + h * HD) = lo;
          *reinterpret_cast<vec4 *>(o + h * HD + 64) = hi;
        }
      }
    }
    return;
  }
  __shared__ f16 tile[64][HD + 2];
  const int h = blockIdx.x % nkv, t0 = blockIdx.x / nkv * 64;
  const float *src = QKV + (int64_t)(heads + h) * HD;
  f32x4 v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int r = k * 8 + (threadIdx.x >> 5), t = t0 + r < n_tok ? t0 + r : n_tok - 1;
    v[k] = *reinterpret_cast<const f32x4 *>(src + (int64_t)t * row + (threadIdx.x & 31) * 4);
  }
  const int t = t0 + lane, col = t < n_tok ? vt_col[t] : 0;
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      tile[k * 8 + (threadIdx.x >> 5)][(threadIdx.x & 31) * 4 + q] = from_f32<f16>(to_f32(from_f32<T>(v[k][q])));
  __syncthreads();
  if (t >= n_tok) return;
  f16 *dst = Vt + (int64_t)h * HD * vt_stride + col;
#pragma unroll 8
  for (int d = wave; d < HD; d += 4) dst[(int64_t)d * vt_stride] = tile[lane][d];
}

// The same in place for the fp32 mode where a head's pairs fit a power of two of lanes (head sizes 32, 64 and 128): P lanes per
// token, so that no lane idles, each with the same pair of up to U heads, their loads issued together; one rotation serves all
// of them, from the table or, where there is none (a call of its own), evaluated while the loads are on their way.  One wave per
// workgroup: a few hundred tokens then reach most compute units.  The sum of squares keeps wave_sum's order (lanes beyond P
// added zeros).  6 heads of 64, a call of its own: 12859 tokens 4.8 (table) + 11.2 us -> 12.0, 354 tokens 2.6 + 2.8 us and the gap
// between them -> 5.1.  Heads beyond U take further blocks, which read the rotations again: with a table, against a lane per pair and head,
// 50 000 tokens of 9 heads of 32 24.6 -> 20.4 us, 24 of 128 286 -> 251, 40 of 128 477 -> 412, 40 of 64 230 -> 237 (the one slower of 120 timed).
template <int P, int U>
__global__ __launch_bounds__(64) void qk_finish_fp32_kernel(float *__restrict__ QKV, const int32_t *__restrict__ pos,
                                                            const float *__restrict__ q_gain, const float *__restrict__ k_gain, int n_tok,
                                                            int nq, int nkv, float eps, int qk_norm, const float2 *__restrict__ rope_tab,
                                                            double log2_base) {
  constexpr int HD = 2 * P, G = 64 / P;                      // tokens of a workgroup
  const int heads = nq + nkv, i = threadIdx.x % P, h0 = blockIdx.y * U;
  const int tw = blockIdx.x * G + threadIdx.x / P, t = tw < n_tok ? tw : n_tok - 1;
  float *x = QKV + (int64_t)t * (nq + 2 * nkv) * HD + i;
  const int p = pos[t];
  float a[U], b[U], gq[2], gk[2];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int h = h0 + u < heads ? h0 + u : heads - 1;
    a[u] = x[h * HD];
    b[u] = x[h * HD + P];
  }
  if (qk_norm) {
    gq[0] = q_gain[i];
    gq[1] = q_gain[i + P];
    gk[0] = k_gain[i];
    gk[1] = k_gain[i + P];
  }
  const float2 cs = rope_tab ? rope_tab[(int64_t)p * P + i] : rotation(p, i, P, log2_base);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int h = h0 + u;
    if (h >= heads) break;                                   // the same for the whole wave
    if (qk_norm) {
      float ss = __builtin_fmaf(a[u], a[u], b[u] * b[u]);
#pragma unroll
      for (int o = P / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
      const float r = 1.0f / sqrtf(ss / (float)HD + eps);
      a[u] = a[u] * r * (h < nq ? gq[0] : gk[0]);
      b[u] = b[u] * r * (h < nq ? gq[1] : gk[1]);
    }
    if (tw < n_tok) {
      x[h * HD] = __builtin_fmaf(a[u], cs.x, -(b[u] * cs.y));
      x[h * HD + P] = __builtin_fmaf(b[u], cs.x, a[u] * cs.y);
    }
  }
}

bool qk_finish_fp32_tiled(int hd) { return hd == 32 || hd == 64 || hd == 128; }

int launch_qk_finish_fp32(float *QKV, const int32_t *pos, const void *q_gain, const void *k_gain, int T, int nq, int nkv, int hd,
                          float eps, int qk_norm, const float2 *rope_tab, float rope_base, hipStream_t s) {
  PRISM_REQUIRE(QKV && pos && (rope_tab || (qk_finish_fp32_tiled(hd) && rope_base > 0)) && T >= 0 && nq > 0 && nkv > 0 && hd > 0 && hd % 2 == 0,
                PRISM_EINVAL, "qk_finish: bad arguments");
  PRISM_REQUIRE(!qk_norm || (q_gain && k_gain), PRISM_EINVAL, "qk_finish: gains missing");
  if (T == 0) return PRISM_OK;
  auto run = [&](auto p) {
    constexpr int P = decltype(p)::value, U = 6;
    qk_finish_fp32_kernel<P, U><<<dim3(cdiv(T, 64 / P), cdiv(nq + nkv, U)), 64, 0, s>>>(QKV, pos, (const float *)q_gain, (const float *)k_gain, T, nq,
                                                                                     nkv, eps, qk_norm, rope_tab, log2((double)rope_base));
  };
  if (hd == 32) run(std::integral_constant<int, 16>{});
  else if (hd == 64) run(std::integral_constant<int, 32>{});
  else if (hd == 128) run(std::integral_constant<int, 64>{});
  else qk_finish_kernel<float><<<cdiv((int64_t)T * (nq + nkv), 4), 256, 0, s>>>(QKV, pos, (const float *)q_gain, (const float *)k_gain, T, nq, nkv, hd,
                                                                            eps, qk_norm, rope_tab, QKV, (nq + 2 * nkv) * hd);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// V part of the fp32 projection -> Vt [nkv][hd][vt_stride], column vt_col[t]: the P V contraction runs
// over keys, so the MFMA operand wants keys contiguous.  P V always runs on the f16 matrix-core
// instruction (the probabilities keep 11 significand bits), so Vt is IEEE half; in bf16-operand mode
// the values are rounded to bf16 first (half holds every bf16 value of normal half range exactly).
// Tile of 64 tokens x hd through LDS.  Serves head sizes other than 128 (and unaligned buffers).
template <typename OT>
__global__ __launch_bounds__(256) void v_finish_kernel(const float *__restrict__ QKV, int n_tok, int nq, int nkv, int hd,
                                                       f16 *__restrict__ Vt, const int32_t *__restrict__ vt_col,
                                                       int64_t vt_stride) {
  __shared__ f16 tile[64][128 + 2];
  const int t0 = blockIdx.x * 64, h = blockIdx.y;
  const int row_elems = (nq + 2 * nkv) * hd;
  const float *src = QKV + (int64_t)(nq + nkv + h) * hd;
  for (int idx = threadIdx.x; idx < 64 * hd; idx += 256) {
    const int r = idx / hd, d = idx % hd;
    if (t0 + r < n_tok) tile[r][d] = from_f32<f16>(to_f32(from_f32<OT>(src[(int64_t)(t0 + r) * row_elems + d])));
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 64 * hd; idx += 256) {
    const int d = idx / 64, r = idx % 64;
    if (t0 + r < n_tok) Vt[((int64_t)h * hd + d) * vt_stride + vt_col[t0 + r]] = tile[r][d];
  }
}

bool qkv_finish_16_direct(const void *QKV, const void *q_gain, const void *k_gain, int hd, int qk_norm, const void *QK) {
  return hd == 128 && (uintptr_t)QKV % 16 == 0 && ((uintptr_t)QK | (qk_norm ? (uintptr_t)q_gain | (uintptr_t)k_gain : 0)) % 8 == 0;
}

int launch_qkv_finish_16(int dtype, const float *QKV, const int32_t *pos, const void *q_gain, const void *k_gain, int T, int nq, int nkv,
                         int hd, float eps, int qk_norm, const float2 *rope_tab, float rope_base, void *QK, void *Vt, const int32_t *vt_col,
                         int64_t vt_stride, hipStream_t s) {
  const bool direct = qkv_finish_16_direct(QKV, q_gain, k_gain, hd, qk_norm, QK);
  PRISM_REQUIRE(QKV && pos && (direct ? rope_base > 0 : rope_tab != nullptr) && QK && Vt && vt_col && T >= 0 && nq > 0 && nkv > 0 && is16(dtype) && hd > 0 && hd <= 128, PRISM_EINVAL,
                "qkv_finish: bad arguments");
  PRISM_REQUIRE(!qk_norm || (q_gain && k_gain), PRISM_EINVAL, "qk_finish: gains missing");
  if (T == 0) return PRISM_OK;
  auto run = [&](auto tag) {
    typedef decltype(tag) OT;
    const OT *gq = (const OT *)q_gain, *gk = (const OT *)k_gain;
    // one launch where every access of four values is aligned; otherwise value by value, by the table
    if (direct) {
      auto go = [&](auto few) {
        constexpr bool kFew = decltype(few)::value;
        qkv_finish_16_kernel<OT, kFew><<<cdiv(T, 64) * nkv + cdiv(T, kFew ? 16 : 4), 256, 0, s>>>(QKV, pos, gq, gk, T, nq, nkv, eps, qk_norm,
                                                                                                log2((double)rope_base), (OT *)QK, (f16 *)Vt, vt_col, vt_stride);
      };
      if (nq + nkv <= 6 && T >= 8192) go(std::true_type{});
      else go(std::false_type{});
      return;
    }
    qk_finish_kernel<OT><<<cdiv((int64_t)T * (nq + nkv), 4), 256, 0, s>>>(const_cast<float *>(QKV), pos, gq, gk, T, nq, nkv, hd, eps, qk_norm, rope_tab,
                                                                          (OT *)QK, (nq + nkv) * hd);
    v_finish_kernel<OT><<<dim3(cdiv(T, 64), nkv), 256, 0, s>>>(QKV, T, nq, nkv, hd, (f16 *)Vt, vt_col, vt_stride);
  };
  if (dtype == PRISM_DTYPE_BF16) run(bf16{});
  else run(f16{});
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// Intermediate scorer (Sec. 4.1): last-token state -> final RMSNorm -> yes/no head rows.
// One workgroup per live candidate; reads H floats; latency-bound.
template <typename T>
__global__ __launch_bounds__(256) void score_kernel(const float *__restrict__ X, const int32_t *__restrict__ last_row,
                                                    int hidden, const T *__restrict__ gain, const T *__restrict__ w_yes,
                                                    const T *__restrict__ w_no, float eps, float *__restrict__ scores) {
  __shared__ float red[4];
  const float *x = X + (int64_t)(last_row ? last_row[blockIdx.x] : (int)blockIdx.x) * hidden;   // no list: state c is row c
  float ss = 0.f, dy = 0.f, dn = 0.f;
#pragma unroll 8
  for (int i = threadIdx.x; i < hidden; i += 256) {          // unrolled: the loads of eight steps are in flight together
    const float v = x[i];
    ss += v * v;
    const float z = v * to_f32(gain[i]);
    dy += z * to_f32(w_yes[i]);
    dn += z * to_f32(w_no[i]);
  }
  ss = block_sum_256(ss, red);
  dy = block_sum_256(dy, red);
  dn = block_sum_256(dn, red);
  if (threadIdx.x == 0) {
    const float r = 1.0f / sqrtf(ss / (float)hidden + eps);
    scores[blockIdx.x] = dy * r - dn * r;
  }
}

int launch_score(const float *X, const int32_t *last_row, int n, int hidden, const void *final_norm,
                 const void *w_yes, const void *w_no, int dtype, float eps, float *scores, hipStream_t s) {
  PRISM_REQUIRE(X && final_norm && w_yes && w_no && scores && n >= 0 && hidden > 0, PRISM_EINVAL, "score: bad arguments");
  if (n == 0) return PRISM_OK;
  if (dtype == PRISM_DTYPE_FP32)
    score_kernel<float><<<n, 256, 0, s>>>(X, last_row, hidden, (const float *)final_norm, (const float *)w_yes,
                                           (const float *)w_no, eps, scores);
  else
    score_kernel<bf16><<<n, 256, 0, s>>>(X, last_row, hidden, (const bf16 *)final_norm, (const bf16 *)w_yes,
                                          (const bf16 *)w_no, eps, scores);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// Compaction (Sec. 4.1: continue only on the remaining candidates): each kept sequence's rows move
// to their new offset in a second buffer, order preserved.  HBM-bound: 2 * T' * H * 4 bytes.  A block moves 16 KiB pieces of its
// sequence, four 16-byte loads per lane in flight, past the caches (neither copy is read again soon): 4.65 -> 4.97 TB/s on
// 109 sequences of 1 GB in all, where a large plain copy reaches 4.67.
__global__ __launch_bounds__(256) void compact_kernel(const float *__restrict__ Xs, float *__restrict__ Xd,
                                                      const int32_t *__restrict__ src_start,
                                                      const int32_t *__restrict__ dst_start,
                                                      const int32_t *__restrict__ len, int hidden) {
  const int c = blockIdx.x, h4 = hidden / 4;
  const int64_t total = (int64_t)len[c] * h4;
  const f32x4 *src = reinterpret_cast<const f32x4 *>(Xs) + (int64_t)src_start[c] * h4;
  f32x4 *dst = reinterpret_cast<f32x4 *>(Xd) + (int64_t)dst_start[c] * h4;
  for (int64_t at = (int64_t)blockIdx.y * 1024 + threadIdx.x; at < total; at += (int64_t)gridDim.y * 1024) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (at + u * 256 < total) v[u] = __builtin_nontemporal_load(src + at + u * 256);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (at + u * 256 < total) __builtin_nontemporal_store(v[u], dst + at + u * 256);
  }
}

int launch_compact(const float *Xs, float *Xd, const int32_t *src_start, const int32_t *dst_start,
                   const int32_t *len, int n_keep, int hidden, hipStream_t s) {
  PRISM_REQUIRE(Xs && Xd && Xs != Xd && src_start && dst_start && len && n_keep >= 0 && hidden % 4 == 0, PRISM_EINVAL,
                "compact: bad arguments");
  if (n_keep == 0) return PRISM_OK;
  // enough blocks to cover the memory latency also for a few sequences, not thousands of idle ones for many (64 per sequence
  // measured 4.97 TB/s, 32 4.77, 256 5.00)
  const int per_seq = n_keep >= 2048 ? 8 : n_keep >= 256 ? 16384 / n_keep : 64;
  compact_kernel<<<dim3(n_keep, per_seq), 256, 0, s>>>(Xs, Xd, src_start, dst_start, len, hidden);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// Shared query: the attention kernel reads its V^T columns in whole groups of 16 where they were written; the columns of a last,
// incomplete group are copied into every sequence's column range.  16 lanes per row and sequence.
__global__ __launch_bounds__(256) void vt_prefix_tail_kernel(f16 *__restrict__ Vt, int64_t vt_stride, int rows, int ql,
                                                             const int32_t *__restrict__ seq_col0) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4), col = (ql & ~15) + (threadIdx.x & 15);
  if (row >= rows || vt_column_of_key(col) >= ql) return;                  // the mapping is its own inverse
  f16 *v = Vt + (int64_t)row * vt_stride;
  v[seq_col0[blockIdx.y] + col] = v[col];
}

int launch_vt_prefix_broadcast(void *Vt, int64_t vt_stride, int rows, int ql, const int32_t *seq_col0, int n_seq, hipStream_t s) {
  PRISM_REQUIRE(Vt && seq_col0 && vt_stride > 0 && rows > 0 && ql > 0 && n_seq >= 0, PRISM_EINVAL, "vt prefix broadcast: bad arguments");
  if (n_seq == 0 || ql % 16 == 0) return PRISM_OK;
  vt_prefix_tail_kernel<<<dim3(cdiv(rows, 16), n_seq), 256, 0, s>>>((f16 *)Vt, vt_stride, rows, ql, seq_col0);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// ------------------------------------------------------------------------------------------------
// Final top-K (Sec. 2.1): rank by counting (score descending, lower position first on ties, NaN behind every number).
// Latency- and issue-bound: n^2 comparisons.  16 lanes per entry, 16 entries per workgroup, so the pool spreads over the
// compute units; the scores are read once into LDS, as whole numbers of the same order, in which NaN has a place too: every
// rank below K is written by exactly one entry, whatever the scores are (the host uses the positions as indices).
// 500 entries 37 us (one workgroup, a memory load per comparison) -> 3.6; 4096: 1490 -> 11.
__global__ __launch_bounds__(256) void topk_kernel(const float *__restrict__ scores, const int8_t *__restrict__ tag,
                                                    int want, int n, int K, int32_t *__restrict__ out_pos,
                                                    float *__restrict__ out_scores) {
  // entries whose tag differs from `want` do not take part (tag == nullptr: all take part): 0, below NaN's 1
  __shared__ uint32_t key[PRISM_MAX_CANDS];
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4);
  const float si = scores[i < n ? i : 0];                                      // requested with the rest, not behind the count
  for (int j = threadIdx.x; j < n; j += 256) {
    const float s = scores[j];
    const uint32_t u = __float_as_uint(s == 0.f ? 0.f : s);                    // -0 ties with 0
    const uint32_t k = s != s ? 1u : (u & 0x80000000u ? ~u : u | 0x80000000u);
    key[j] = tag && tag[j] != want ? 0u : k;
  }
  __syncthreads();
  if (i >= n || key[i] == 0u) return;
  const uint32_t ki = key[i];
  int rank = 0;
#pragma unroll 4
  for (int j = threadIdx.x & 15; j < n; j += 16) {
    rank += key[j] > ki - (j < i ? 1u : 0u);                                   // j in front of i also when equal
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 64);
  if ((threadIdx.x & 15) == 0 && rank < K) {
    out_pos[rank] = i;
    out_scores[rank] = si;
  }
}

int launch_topk_masked(const float *scores, const int8_t *tag, int want, int n, int K, int32_t *out_pos,
                       float *out_scores, hipStream_t s) {
  PRISM_REQUIRE(scores && out_pos && out_scores && n >= 0 && K >= 0, PRISM_EINVAL, "topk: bad arguments");
  if (n == 0 || K == 0) return PRISM_OK;
  topk_kernel<<<cdiv(n, 16), 256, 0, s>>>(scores, tag, want, n, K, out_pos, out_scores);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

int launch_topk(const float *scores, int n, int K, int32_t *out_pos, float *out_scores, hipStream_t s) {
  return launch_topk_masked(scores, nullptr, 0, n, K, out_pos, out_scores, s);
}

__global__ void fill_zero_kernel(uint4 *p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

// Copies between pinned host memory and the device as kernels on the compute stream.  A check's results and the metadata rebuilt
// from them are a few KiB to some 100 KiB on the call's critical path; as copies of the runtime they cross to a DMA engine and
// back, and a host that slept until the stream drained wakes late.  From a decision to the next kernel, traced: 37 us -> 14-22
// without a compaction, 67 + 10 -> 59 + 12 with one; with the layers' shared moments six short candidates on the 0.6B shape 2280 -> 2205 us,
// forty of 128-480 tokens 7000 -> 6940.  Accesses on the host's side have system scope, past every cache, since the host rewrites
// the buffers between calls; 8 bytes per lane, the largest such.
//
// host -> device: up to kCopyParts ranges of one pair of buffers (blockIdx.y).
__global__ __launch_bounds__(256) void fetch_host_kernel(const uint64_t *__restrict__ src, uint64_t *__restrict__ dst, const CopyParts parts) {
  const uint32_t first = parts.first[blockIdx.y], n = parts.n[blockIdx.y];
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
    dst[first + i] = __hip_atomic_load(src + first + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// device -> host, in one workgroup, so that its barrier orders the flag behind every word.
__global__ __launch_bounds__(1024) void post_host_kernel(const uint64_t *__restrict__ src, const HostPost post) { post_host(src, post); }

int launch_fetch_host(const void *src, void *dst, const CopyParts &parts, hipStream_t s) {
  PRISM_REQUIRE(src && dst && parts.count >= 0 && parts.count <= kCopyParts && ((uintptr_t)src | (uintptr_t)dst) % 8 == 0, PRISM_EINVAL, "host copy: bad arguments");
  uint32_t most = 0;
  for (int i = 0; i < parts.count; ++i) most = parts.n[i] > most ? parts.n[i] : most;
  if (most == 0) return PRISM_OK;
  fetch_host_kernel<<<dim3(cdiv(most, 256) < 64 ? cdiv(most, 256) : 64, parts.count), 256, 0, s>>>((const uint64_t *)src, (uint64_t *)dst, parts);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

int launch_post_host(const void *src, const HostPost &post, hipStream_t s) {
  PRISM_REQUIRE(src && post.dst && post.flag && post.words >= 0 && ((uintptr_t)src | (uintptr_t)post.dst | (uintptr_t)post.flag) % 8 == 0, PRISM_EINVAL,
                "host copy: bad arguments");
  post_host_kernel<<<1, 1024, 0, s>>>((const uint64_t *)src, post);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

// In place, 8 elements (16 bytes) per lane and step over the first n8 * 8 elements, one element per lane over the rest.
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(unsigned short *p, size_t n, size_t n8) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  auto half_bits = [](unsigned bf16_in_high_half) -> unsigned {
    const f16 h = from_f32<f16>(__uint_as_float(bf16_in_high_half));
    return (unsigned)*reinterpret_cast<const unsigned short *>(&h);
  };
  uint4 *q = reinterpret_cast<uint4 *>(p);
  for (size_t i = t; i < n8; i += stride) {
    const uint4 v = q[i];
    unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = half_bits(w[k] << 16) | (half_bits(w[k] & 0xffff0000u) << 16);
    q[i] = make_uint4(w[0], w[1], w[2], w[3]);
  }
  for (size_t i = n8 * 8 + t; i < n; i += stride) p[i] = (unsigned short)half_bits((unsigned)p[i] << 16);
}

int launch_bf16_to_f16(void *p, size_t n, hipStream_t s) {
  PRISM_REQUIRE(p, PRISM_EINVAL, "bf16_to_f16: null pointer");
  if (n == 0) return PRISM_OK;
  const size_t n8 = (reinterpret_cast<uintptr_t>(p) % 16 == 0) ? n / 8 : 0;      // 16-byte steps need a 16-byte aligned buffer
  const size_t work = n8 ? n8 : n, blocks = (work + 255) / 256;
  bf16_to_f16_kernel<<<(int)(blocks < 8192 ? blocks : 8192), 256, 0, s>>>((unsigned short *)p, n, n8);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

int launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
  PRISM_REQUIRE(p && bytes % 16 == 0, PRISM_EINVAL, "fill_zero: bad arguments");
  if (bytes == 0) return PRISM_OK;
  const size_t n16 = bytes / 16;
  const int grid = (int)((n16 + 255) / 256 < 4096 ? (n16 + 255) / 256 : 4096);
  fill_zero_kernel<<<grid, 256, 0, s>>>((uint4 *)p, n16);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

}  // namespace prism
