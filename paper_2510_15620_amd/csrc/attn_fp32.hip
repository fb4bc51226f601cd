// Causal GQA attention for the fp32 mode.
//
// attention_fp32_kernel: head sizes 32, 64 and 128, on v_mfma_f32_16x16x4_f32.  A wavefront owns 16 queries of one head, its
// workgroup 64 consecutive queries of one sequence (a work item); the waves share nothing and meet at no barrier (LDS holds the
// values of each wave's own diagonal tile).  As in the 16-bit
// kernel everything is computed transposed, S^T = K Q^T and O^T += V^T P^T, so that a lane owns one query (lane % 16) and
// the accumulators of S^T are the next contraction's operand as they are: instruction s of the second contraction takes
// the four keys 4 g + s, g = 0..3, and a lane of group g = lane / 16 holds the weight of key 4 g + s in register s.  Operands
// come straight from memory in 16-byte pieces (K: four consecutive dimensions of a key; V: NB consecutive dimensions, which
// become the same row of the NB accumulator tiles), one tile of 16 keys ahead; the four waves of a workgroup and the heads of a
// group meet in L1 and L2.  Bound by the chain of a tile (32 NB / 4 matrix instructions, softmax) with few waves per SIMD.
// The tile on the diagonal, the only one with masked keys, takes its P V part on the vector pipes under the mask: a weight of
// zero times a non-finite value of a token in the future would otherwise reach the sum.  Until a query has met a finite score
// its running maximum is -inf and its weights are taken relative to 0, so leading keys that score -inf weigh nothing.  Partial
// sums of values have weights of up to 1 per key, so values need to stay below the largest fp32 number over the sequence length.
// 4 heads of 64, 12859 tokens of 160-512-token sequences: 771 us as one workgroup per (token, head) -> 86 us; -> 79 with the next
// tile's loads held in front of a tile's work, the accumulators in vector registers and the diagonal's values handed over in LDS;
// -> 55 with the items longest first (attention_fp32_longest_first).  8 sequences of 32-64 tokens 11.2 -> 8.5.
//
// attention_fp32_any_kernel: any other head size: the definition, one workgroup per (token, query head), score row in LDS.
#include "common.h"

namespace prism {

template <int NB, typename Items>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NB <= 4 ? 3 : 2))) void attention_fp32_kernel(const float *__restrict__ QKV, const Items items,
                                                             int nq, int nkv, float *__restrict__ out) {
  constexpr int HD = 16 * NB;
  __shared__ __align__(16) float diag[4 * 16 * HD];          // per wave: the values of its diagonal tile
  const AttnTile it = items(blockIdx.x / nq);
  const int h = blockIdx.x % nq, kvh = h / (nq / nkv);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int L = it.seq_len, q0 = it.q0 + wave * 16;
  if (q0 >= L) return;
  const int64_t row = (int64_t)(nq + 2 * nkv) * HD;
  const float *base = QKV + (int64_t)it.row_base * row;
  const float *kcol = base + (int64_t)(nq + kvh) * HD + 4 * g, *vcol = base + (int64_t)(nq + nkv + kvh) * HD;
  const int qi = q0 + c < L ? q0 + c : L - 1;                // this lane's query (the last one again where there are fewer)
  f32x4 qf[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) qf[b] = *reinterpret_cast<const f32x4 *>(base + (int64_t)qi * row + (int64_t)h * HD + 16 * b + 4 * g);

  struct Tile { f32x4 k[NB]; float v[4][NB]; };
  auto fetch = [&](int k0, Tile &t) __attribute__((always_inline)) {
    const float *kp = kcol + (int64_t)(k0 + c < L ? k0 + c : L - 1) * row;
#pragma unroll
    for (int b = 0; b < NB; ++b) t.k[b] = *reinterpret_cast<const f32x4 *>(kp + 16 * b);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int key = k0 + 4 * g + s;
      const float *vp = vcol + (int64_t)(key < L ? key : L - 1) * row + NB * c;
      if constexpr (NB == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(vp);
        t.v[s][0] = v.x; t.v[s][1] = v.y;
      } else {
#pragma unroll
        for (int j = 0; j < NB; j += 4) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(vp + j);
          t.v[s][j] = v[0]; t.v[s][j + 1] = v[1]; t.v[s][j + 2] = v[2]; t.v[s][j + 3] = v[3];
        }
      }
    }
  };

  f32x4 o[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float scale = 1.0f / sqrtf((float)HD);

  // scores of one tile of keys, running maximum, weights: p[s] is the weight of key k0 + 4 g + s
  auto weigh = [&](int k0, const Tile &t, bool masked, float *p) __attribute__((always_inline)) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; b += 2)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[b][s], qf[b][s], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[b + 1][s], qf[b + 1][s], s1, 0, 0, 0);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      p[s] = (s0[s] + s1[s]) * scale;
      if (masked && k0 + 4 * g + s > qi) p[s] = -INFINITY;
      mx = fmaxf(mx, p[s]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float ref = m_new == -INFINITY ? 0.f : m_new;      // all keys so far score -inf: weights exp(-inf) = 0, not exp(-inf + inf)
    const float alpha = expf(m_run - ref);
    m_run = m_new;
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      p[s] = expf(p[s] - ref);
      sum += p[s];
    }
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int b = 0; b < NB; ++b) o[b] *= alpha;
  };

  float p[4];
  auto past = [&](int k0, const Tile &t) __attribute__((always_inline)) {      // a tile whose keys are all in every query's past
    weigh(k0, t, false, p);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int b = 0; b < NB; ++b) o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.v[s][b], p[s], o[b], 0, 0, 0);
  };
  // Two tiles' registers in turn.  The scheduling barriers keep a tile's loads in front of the work on the tile before: without
  // them the compiler moves them behind it to save registers, and every tile waits for memory.
  Tile cur, next;
  fetch(0, cur);
  int k0 = 0;
  for (; k0 + 32 <= q0; k0 += 32) {
    fetch(k0 + 16, next);
    __builtin_amdgcn_sched_barrier(0);
    past(k0, cur);
    fetch(k0 + 32, cur);
    __builtin_amdgcn_sched_barrier(0);
    past(k0 + 16, next);
  }
  if (k0 < q0) {
    fetch(k0 + 16, next);
    __builtin_amdgcn_sched_barrier(0);
    past(k0, cur);
    cur = next;
  }
  weigh(q0, cur, true, p);
  // the diagonal tile: o[b][e] is dimension NB (4 g + e) + b of query lane % 16.  A lane needs 4 NB dimensions of every key here; the
  // wave has the tile's values, other dimensions of four keys in a lane, and hands them over through LDS of its own
  float *vd = diag + (threadIdx.x >> 6) * (16 * HD);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < NB; ++j) vd[(4 * g + s) * HD + NB * c + j] = cur.v[s][j];
  // (LDS serves a wave in order; the fences keep the compiler to it, the barrier, no instruction, makes the lanes meet)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int k0 = 0; k0 < 16 && q0 + k0 < L; k0 += 4) {
    f32x4 v[4][NB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < NB; ++j) v[u][j] = *reinterpret_cast<const f32x4 *>(vd + (k0 + u) * HD + NB * 4 * g + 4 * j);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float w = __shfl(p[u], k0 * 4 + c);              // key k0 + u: register u of group k0 / 4
      if (q0 + k0 + u <= qi) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) o[(4 * j + q) % NB][(4 * j + q) / NB] += w * v[u][j][q];
      }
    }
  }
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (q0 + c >= L) return;
  float *op = out + ((int64_t)(it.out_base + qi) * nq + h) * HD + NB * 4 * g;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = o[(4 * j + q) % NB][(4 * j + q) / NB] / l_run;
    *reinterpret_cast<f32x4 *>(op + 4 * j) = v;
  }
}

__global__ __launch_bounds__(128) void attention_fp32_any_kernel(const float *__restrict__ QKV,
                                                             const int32_t *__restrict__ pos, int nq, int nkv, int hd,
                                                             float *__restrict__ out) {
  extern __shared__ float p[];          // [pos + 1] scores, then [hd] the query
  __shared__ float red[2];
  const int t = blockIdx.x, h = blockIdx.y;
  const int i = pos[t], n_keys = i + 1;
  const int row = (nq + 2 * nkv) * hd, kvh = h / (nq / nkv);
  const float *q = QKV + (int64_t)t * row + (int64_t)h * hd;
  const float *kbase = QKV + (int64_t)(t - i) * row + (int64_t)(nq + kvh) * hd;
  const float *vbase = kbase + (int64_t)nkv * hd;
  float *qs = p + n_keys;
  for (int d = threadIdx.x; d < hd; d += 128) qs[d] = q[d];
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)hd);
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < n_keys; j += 128) {
    const float *k = kbase + (int64_t)j * row;
    float dot = 0.f;
    for (int d = 0; d < hd; ++d) dot += qs[d] * k[d];
    dot *= scale;
    p[j] = dot;
    mx = fmaxf(mx, dot);
  }
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(red[0], red[1]);
  __syncthreads();
  float sum = 0.f;
  for (int j = threadIdx.x; j < n_keys; j += 128) {
    const float e = expf(p[j] - mx);
    p[j] = e;
    sum += e;
  }
  sum = wave_sum(sum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = red[0] + red[1];
  for (int d = threadIdx.x; d < hd; d += 128) {
    float acc = 0.f;
    for (int j = 0; j < n_keys; ++j) acc += p[j] * vbase[(int64_t)j * row + d];
    out[(int64_t)t * nq * hd + (int64_t)h * hd + d] = acc / sum;
  }
}

bool attention_fp32_tiled(int hd) { return hd == 32 || hd == 64 || hd == 128; }

// The order of a launch's items.  Longest first evens out the compute units' shares, worth up to 40 % while a unit gets few items, but
// keeps every sequence's K/V in use from the first item to the last.  Sequence by sequence only a few are: that wins, by up to 30 %, once
// the pool's K/V are more than the caches hold, the earlier the more heads read them on different XCDs.  Over 267 pools (14 000 to 360 000
// tokens of sequences of 60 to 8192, 2 to 32 query heads of 32 to 128) the rule's order is on average 0.4 % behind the faster one (always
// longest first 1.4 %, never 7.4 %) and at worst 7 %, but for one pool of equal lengths (100 of 512, 16 / 16 heads of 32: a unit is dealt the
// same block of every sequence; ms by sequence 0.447, longest first 0.394).  ms likewise, 16 / 8 heads of 64: 14 065 tokens 0.179,
// 0.158; 45 907 of 512-1024 0.93, 0.99; 327 680 of 8192 57.1, 74.8; 8 / 8 heads of 64: 64 624 of 288-1024 0.64, 0.59; 362 962 of 200-512 2.22, 2.36.
bool attention_fp32_longest_first(int64_t tokens, int nq, int nkv, int hd) {
  const int64_t kv_bytes = tokens * nkv * hd * 8;
  return kv_bytes <= (nq <= 12 ? 512000000 : 128000000);
}

template <typename Items>
static int launch_items(const float *QKV, const Items &items, int n_tiles, int nq, int nkv, int hd, float *out, hipStream_t s) {
  if (n_tiles == 0) return PRISM_OK;
  PRISM_REQUIRE((int64_t)n_tiles * nq < (int64_t)1 << 31, PRISM_EINVAL, "attention: too many work items (%d x %d)", n_tiles, nq);
  const int grid = n_tiles * nq;
  if (hd == 32) attention_fp32_kernel<2><<<grid, 256, 0, s>>>(QKV, items, nq, nkv, out);
  else if (hd == 64) attention_fp32_kernel<4><<<grid, 256, 0, s>>>(QKV, items, nq, nkv, out);
  else attention_fp32_kernel<8><<<grid, 256, 0, s>>>(QKV, items, nq, nkv, out);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

int launch_attention_fp32_levels(const float *QKV, const AttnLevels &levels, int nq, int nkv, int hd, float *out, hipStream_t s) {
  PRISM_REQUIRE(QKV && out && nq > 0 && nkv > 0 && nq % nkv == 0 && attention_fp32_tiled(hd) && ((uintptr_t)QKV | (uintptr_t)out) % 16 == 0 &&
                levels.n_levels > 0 && levels.n_levels <= PRISM_MAX_SEQ / kAttn32BQ, PRISM_EINVAL, "attention fp32: bad arguments");
  return launch_items(QKV, levels, levels.end[levels.n_levels - 1], nq, nkv, hd, out, s);
}

int launch_attention_fp32(const float *QKV, const int32_t *pos, const AttnTile *tiles, int n_tiles, int T, int nq, int nkv, int hd, float *out,
                          hipStream_t s) {
  PRISM_REQUIRE(QKV && out && T >= 0 && nq > 0 && nkv > 0 && nq % nkv == 0 && hd > 0, PRISM_EINVAL,
                "attention fp32: bad arguments");
  if (T == 0) return PRISM_OK;
  if (tiles && attention_fp32_tiled(hd) && ((uintptr_t)QKV | (uintptr_t)out) % 16 == 0)
    return launch_items(QKV, AttnList{tiles}, n_tiles, nq, nkv, hd, out, s);
  PRISM_REQUIRE(pos, PRISM_EINVAL, "attention fp32: bad arguments");
  const size_t lds = (size_t)(PRISM_MAX_SEQ + hd) * sizeof(float);
  PRISM_REQUIRE(lds <= 64 * 1024, PRISM_EUNSUPPORTED, "attention fp32: head_dim %d too large", hd);
  attention_fp32_any_kernel<<<dim3(T, nq), 128, lds, s>>>(QKV, pos, nq, nkv, hd, out);
  PRISM_HIP(hipGetLastError());
  return PRISM_OK;
}

}  // namespace prism
