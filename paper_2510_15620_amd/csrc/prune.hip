// One pruning check on the live candidates' provisional scores (paper Sec. 4.1, worked example
// Sec. 4.5): dispersion gate on the coefficient of variation, K-Means of the scalar scores, routing
// around the boundary cluster.
//
// The paper runs K-Means on the CPU (~1 ms); here it runs on the device so the scores
// never leave HBM before the decision.  K-Means of scalars is solved exactly: every optimum of the
// within-cluster sum of squares is a partition of the ranked scores into consecutive runs, so a
// dynamic programme over split positions finds it, with no seed and no iteration count.
//
// All decisions are taken in fp64 with a fixed operation order (sequential sums, no fused
// multiply-add: this file is compiled with -ffp-contract=off), so that a host implementation that
// follows the same order reaches the same bits.
#include <algorithm>
#include <mutex>

#include "common.h"

namespace prism {

struct RouteWs {
  double *ranked, *P, *Q, *E0, *E1;
  int32_t *order, *arg;  // arg: [k+1][n+1]
};

__device__ __forceinline__ double run_cost(const double *P, const double *Q, int i, int j) {
  const double sp = P[j] - P[i];
  return (Q[j] - Q[i]) - sp * sp / (double)(j - i);
}

// The decision in four phases.  What bounds them: the sums of the first two are chains of dependent fp64 additions in a
// prescribed order (n of them, about 4 ns each); the table of the third has n^2 / 2 entries per stage, each with an fp64
// division when done plainly.  Small pools (up to kOneGroup) run all phases in one workgroup on LDS; larger ones as
// 2 + (k - 2) launches: phase 1 and 2 side by side on two compute units, the table on all of them, the rest on one.
// us of kernels per call, 3 clusters, sums over floats as they were sorted -> over doubles laid out for them: 12 candidates
// 7.8 -> 7.6, 100: 15.6 -> 14.7, 500: 36 -> 33, 1000: 53 -> 47, 4096: 183 -> 142 (one workgroup on global memory took 53 for 100,
// 232 for 500, 4895 for 4096).  The border between the two forms: 128 candidates, 8 clusters took 41 as one workgroup, 129 took 45
// (launches included, before the sums were changed).

// f(i, x[i]) for i = 0 .. n - 1, in order, by one thread; x in LDS, 16-byte aligned, and already what is summed: one wavefront issues
// its fp64 instructions one after another, so a conversion or a product beside each addition lengthens the chain (the last
// launch on 4096 candidates: 34 us with a conversion from float in it, 23 without).  Sixteen values are read ahead, so that the chain of additions in f is
// all there is to wait for.
template <typename F>
__device__ __forceinline__ void in_order(const double *x, int n, F f) {
  typedef __attribute__((ext_vector_type(2))) double f64x2;
  const f64x2 *q = reinterpret_cast<const f64x2 *>(x);
  int i = 0;
  if (n >= 16) {
    f64x2 cur[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cur[j] = q[j];
    for (; i + 16 <= n; i += 16) {
      f64x2 next[8];
      const int at = i + 32 <= n ? i / 2 + 8 : 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) next[j] = q[at + j];
#pragma unroll
      for (int j = 0; j < 16; ++j) f(i + j, cur[j / 2][j % 2]);
#pragma unroll
      for (int j = 0; j < 8; ++j) cur[j] = next[j];
    }
  }
  for (; i < n; ++i) f(i, x[i]);
}

// ---- phase 1: mean and population std, sequential in index order; the gate.  In two halves, each a chain of one thread, with the
// squared deviations between them by the whole workgroup (deviate).  x is in LDS.
__device__ __forceinline__ double mean_phase(const double *x, int n) {
  double tot = 0.0;
  in_order(x, n, [&](int, double v) { tot = tot + v; });
  return n > 0 ? tot / (double)n : 0.0;
}
__device__ __forceinline__ void deviate(double *x, int n, double mean) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double d = x[i] - mean;
    x[i] = d * d;
  }
}
__device__ __forceinline__ void stats_phase(const double *sq, int n, int K_rem, float tau, double mean, double *stats) {
  double acc = 0.0;
  in_order(sq, n, [&](int, double v) { acc = acc + v; });
  const double sd = n > 0 ? sqrt(acc / (double)n) : 0.0;
  const int gate = (n > K_rem) && (sd > (double)tau * fabs(mean));   // CV > tau, division-free
  stats[0] = mean;
  stats[1] = sd;
  stats[2] = (double)gate;
  stats[3] = 0.0;
}

// ---- phase 2, from the scores in rank order (sorted, in LDS): sequential prefix sums P, Q of x and x^2 (a thread each, in different
// wavefronts; in LDS, so that a sum costs its thread no store to memory), number of clusters, first row of costs
// E[1][i] = cost(i, n).  The whole workgroup.
__device__ void prefix_phase(const float *sorted, int n, int k_req, int *sh_distinct, double *x, double *xx, double *P, double *Q,
                             const RouteWs &ws) {
  const int tid = threadIdx.x, nt = blockDim.x;
  if (tid == 0) *sh_distinct = 0;
  __syncthreads();
  int local = 0;
  for (int r = tid; r < n; r += nt) {
    const double v = (double)sorted[r];
    ws.ranked[r] = x[r] = v;
    xx[r] = v * v;
    local += r == 0 || sorted[r - 1] != sorted[r];
  }
  if (local) atomicAdd(sh_distinct, local);
  __syncthreads();
  double run = 0.0;
  if (tid == 0) {
    P[0] = 0.0;
    in_order(x, n, [&](int i, double v) { P[i + 1] = run = run + v; });
  } else if (tid == 64) {
    Q[0] = 0.0;
    in_order(xx, n, [&](int i, double v) { Q[i + 1] = run = run + v; });
  }
  __syncthreads();
  for (int i = tid; i < n; i += nt) ws.E0[i] = run_cost(P, Q, i, n);
  if (tid == 0) ws.arg[0] = k_req < *sh_distinct ? k_req : *sh_distinct;       // row 0 of the split table is not used otherwise
  __syncthreads();
}

// Order of a large pool: score descending, lower index first on ties, by a bitonic sort of (score, index) keys in LDS; the
// scores are left in rank order.  A pool whose gate is open holds finite scores only (an infinity or NaN makes the std NaN), so
// the key order is the order of the scores.
__device__ void sort_phase(float *sc, int n, unsigned long long *key, const RouteWs &ws) {
  const int tid = threadIdx.x, nt = blockDim.x;
  int np = 2;
  while (np < n) np *= 2;
  for (int i = tid; i < np; i += nt) {
    unsigned long long v = ~0ull;
    if (i < n) {
      const float s = sc[i] == 0.f ? 0.f : sc[i];                              // -0 ties with 0
      const unsigned u = __float_as_uint(s);
      v = (unsigned long long)(u & 0x80000000u ? u : ~(u | 0x80000000u)) << 32 | (unsigned)i;   // larger score, smaller key
    }
    key[i] = v;
  }
  __syncthreads();
  for (int size = 2; size <= np; size *= 2)
    for (int d = size / 2; d > 0; d /= 2) {
      for (int t = tid; t < np / 2; t += nt) {
        const int i = 2 * t - (t & (d - 1)), j = i + d;
        const unsigned long long x = key[i], y = key[j];
        if ((x > y) == ((i & size) == 0)) { key[i] = y; key[j] = x; }
      }
      // pairs up to 64 apart: a wavefront's 64 pairs are the same 128 keys in every such step, and LDS serves it in order.  The
      // barrier of the wavefront (no instruction) is what makes its lanes meet behind the exchange, which each enters or not; the
      // fences order its memory accesses only.
      const int next = d > 1 ? d / 2 : size;
      if (d > 64 || next > 64) __syncthreads();
      else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  __syncthreads();
  float mine[PRISM_MAX_CANDS / 1024];
#pragma unroll
  for (int j = 0; j < PRISM_MAX_CANDS / 1024; ++j) {
    const int r = tid + j * 1024;
    if (r < n) {
      const int i = (int)(key[r] & 0xffffffffu);
      ws.order[r] = i;
      mine[j] = sc[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PRISM_MAX_CANDS / 1024; ++j)
    if (tid + j * 1024 < n) sc[tid + j * 1024] = mine[j];
  __syncthreads();
}

// ---- phase 3: row m of the table: E[m][i] = best cost of cutting ranked[i:] into m runs, split at the smallest s among equal
// costs.  One wavefront per i.  A cost with the division replaced by a single-precision reciprocal is off by at most
// 2^-22 of the pool's sum of squares S (every term of a cost is at most S), so only the s whose approximate cost comes
// within 1e-6 S of the smallest approximate one can be the answer, and only those take the division.
__device__ void table_phase(int m, int n, const RouteWs &ws, int wave, int n_waves) {
  const double *P = ws.P, *Q = ws.Q, *Eprev = m % 2 == 0 ? ws.E0 : ws.E1;
  double *Ecur = m % 2 == 0 ? ws.E1 : ws.E0;
  int32_t *arg = ws.arg + (int64_t)m * (n + 1);
  const int lane = threadIdx.x & 63, last = n - (m - 1);
  const double margin = 1e-6 * Q[n];
  for (int i = wave; i <= n - m; i += n_waves) {
    const double Pi = P[i], Qi = Q[i];
    auto rough = [&](int s) {
      const double sp = P[s] - Pi;
      return (Q[s] - Qi) - sp * sp * (double)__builtin_amdgcn_rcpf((float)(s - i)) + Eprev[s];
    };
    double least = INFINITY;
    for (int s = i + 1 + lane; s <= last; s += 64) {
      const double c = rough(s);
      if (c < least) least = c;
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double c = __shfl_xor(least, o, 64);
      if (c < least) least = c;
    }
    double best = INFINITY;
    int best_s = 0x7fffffff;
    for (int s = i + 1 + lane; s <= last; s += 64) {
      if (rough(s) > least + margin) continue;
      const double c = run_cost(P, Q, i, s) + Eprev[s];
      if (c < best) { best = c; best_s = s; }
    }
    for (int o = 32; o > 0; o >>= 1) {
      const double c = __shfl_xor(best, o, 64);
      const int s = __shfl_xor(best_s, o, 64);
      if (c < best || (c == best && s < best_s)) { best = c; best_s = s; }
    }
    if (lane == 0) {
      Ecur[i] = best;
      arg[i] = best_s;
    }
  }
}

// ---- phase 4: the last stage is only needed at i = 0; then the split positions, cluster means (sequential sums, a thread per
// cluster), the boundary cluster and the fates.  The whole workgroup (up to 1024 threads).
struct RouteShared {
  double val[16];
  int idx[16], splits[PRISM_MAX_CLUSTERS + 1], b;
  double means[PRISM_MAX_CLUSTERS];
};
__device__ void fate_phase(int k, int n, int K_rem, int8_t *fate, double *stats, const double *ranked, const RouteWs &ws, RouteShared &sh) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const double *Eprev = k % 2 == 0 ? ws.E0 : ws.E1;
  double best = INFINITY;
  int best_s = 0x7fffffff;
  for (int s = 1 + tid; s <= n - (k - 1); s += nt) {
    const double c = run_cost(ws.P, ws.Q, 0, s) + Eprev[s];
    if (c < best) { best = c; best_s = s; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double c = __shfl_xor(best, o, 64);
    const int s = __shfl_xor(best_s, o, 64);
    if (c < best || (c == best && s < best_s)) { best = c; best_s = s; }
  }
  if (lane == 0) { sh.val[wave] = best; sh.idx[wave] = best_s; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < (nt >> 6); ++w)
      if (sh.val[w] < best || (sh.val[w] == best && sh.idx[w] < best_s)) { best = sh.val[w]; best_s = sh.idx[w]; }
    sh.splits[0] = 0;
    int i = best_s;
    sh.splits[1] = i;
    for (int m = k - 1, c = 2; m >= 2; --m, ++c) {
      i = ws.arg[(int64_t)m * (n + 1) + i];
      sh.splits[c] = i;
    }
    sh.splits[k] = n;
    int b = 0;
    for (int c = 0; c < k; ++c)
      if (sh.splits[c] <= K_rem - 1 && K_rem - 1 < sh.splits[c + 1]) b = c;
    sh.b = b;
    stats[3] = (double)k;
  }
  __syncthreads();
  if (lane == 0)
  for (int cl = wave; cl < k; cl += nt >> 6) {               // a cluster per wavefront
    const int from = sh.splits[cl], to = sh.splits[cl + 1];
    double tot = 0.0;
    int r = from;
    for (; r < to && r % 2 != 0; ++r) tot = tot + ranked[r];
    in_order(ranked + r, to - r, [&](int, double v) { tot = tot + v; });
    sh.means[cl] = tot / (double)(to - from);
  }
  __syncthreads();
  const double mb = sh.means[sh.b];
  for (int r = tid; r < n; r += nt) {
    int c = 0;
    while (r >= sh.splits[c + 1]) ++c;
    const double mc = sh.means[c];
    fate[ws.order[r]] = mc > mb ? PRISM_FATE_SELECTED : (mc < mb ? PRISM_FATE_DROPPED : PRISM_FATE_DEFERRED);
  }
}

static constexpr int kOneGroup = 128;

// everything in one workgroup, n <= kOneGroup: rank by counting and the plain costs, 4 and 16 lanes per candidate
__device__ __forceinline__ void route_small(const float *__restrict__ scores, int n, int K_rem, int k_req, float tau, int8_t *fate, double *stats) {
  __shared__ __align__(16) float sc[kOneGroup], sorted[kOneGroup];
  __shared__ __align__(16) double arr[5][kOneGroup + 2], x[kOneGroup], xx[kOneGroup];
  __shared__ int32_t order[kOneGroup], arg[(PRISM_MAX_CLUSTERS + 1) * (kOneGroup + 1)];
  __shared__ double st[4];
  __shared__ int distinct;
  __shared__ RouteShared sh;
  const RouteWs ws{arr[0], arr[1], arr[2], arr[3], arr[4], order, arg};
  const int tid = threadIdx.x;
  if (tid < n) {
    sc[tid] = scores[tid];
    x[tid] = (double)scores[tid];
    fate[tid] = PRISM_FATE_DEFERRED;
  }
  __syncthreads();
  {
    const int i = tid >> 2;                                  // ranks while thread 0 of the last wavefront sums
    const float si = i < n ? sc[i] : 0.f;
    int r = 0;
    for (int j = tid & 3; j < n; j += 4) {
      const float sj = sc[j];
      r += (sj > si) || (sj == si && j < i);
    }
    r += __shfl_xor(r, 1, 64);
    r += __shfl_xor(r, 2, 64);
    if (i < n && (tid & 3) == 0) {
      order[r] = i;
      sorted[r] = si;
    }
  }
  if (tid == 511) st[0] = mean_phase(x, n);
  __syncthreads();
  deviate(x, n, st[0]);
  __syncthreads();
  if (tid == 511) stats_phase(x, n, K_rem, tau, st[0], st);
  __syncthreads();
  if (tid < 4) stats[tid] = st[tid];
  if (st[2] == 0.0) return;
  prefix_phase(sorted, n, k_req, &distinct, x, xx, ws.P, ws.Q, ws);
  const int k = arg[0];
  if (k <= 1) return;
  for (int m = 2; m < k; ++m) {
    const double *Eprev = m % 2 == 0 ? ws.E0 : ws.E1;
    double *Ecur = m % 2 == 0 ? ws.E1 : ws.E0;
    for (int i = tid >> 4; i <= n - m; i += 32) {
      double best = INFINITY;
      int best_s = 0x7fffffff;
      for (int s = i + 1 + (tid & 15); s <= n - (m - 1); s += 16) {
        const double c = run_cost(ws.P, ws.Q, i, s) + Eprev[s];
        if (c < best) { best = c; best_s = s; }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const double c = __shfl_xor(best, o, 64);
        const int s = __shfl_xor(best_s, o, 64);
        if (c < best || (c == best && s < best_s)) { best = c; best_s = s; }
      }
      if ((tid & 15) == 0) {
        Ecur[i] = best;
        arg[m * (n + 1) + i] = best_s;
      }
    }
    __syncthreads();
  }
  fate_phase(k, n, K_rem, fate, stats, ws.ranked, ws, sh);
}

// The one workgroup that decides also posts the result block to the host where it is asked to (post.flag; the block starts with
// stats): a launch of its own for that took 5 us on the
// way from the scores to the host's next launch (six short candidates on the 0.6B shape, six checks: 2216 -> 2201 us).  What it posts was
// stored as doubles and bytes, by other lanes too: the barrier in between is what puts those stores in front of the words' loads.
__global__ __launch_bounds__(512) void route_small_kernel(const float *__restrict__ scores, int n, int K_rem, int k_req, float tau,
                                                          int8_t *fate, double *stats, const HostPost post) {
  route_small(scores, n, K_rem, k_req, tau, fate, stats);
  if (!post.flag) return;
  __syncthreads();
  post_host(reinterpret_cast<const uint64_t *>(stats), post);
}

// n > kOneGroup.  Block 0: phase 1 and the default fates; block 1: phase 2 (wasted when the gate turns out closed).
__global__ __launch_bounds__(1024) void route_prepare_kernel(const float *__restrict__ scores, int n, int K_rem, int k_req, float tau,
                                                             int8_t *__restrict__ fate, double *__restrict__ stats, RouteWs ws) {
  // (xx is the sort's key array first)
  __shared__ __align__(16) float sc[PRISM_MAX_CANDS];
  __shared__ __align__(16) double x[PRISM_MAX_CANDS], xx[PRISM_MAX_CANDS], P[PRISM_MAX_CANDS + 1], Q[PRISM_MAX_CANDS + 1];
  __shared__ int distinct;
  __shared__ double mean;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    sc[i] = scores[i];
    x[i] = (double)scores[i];
    if (blockIdx.x == 0) fate[i] = PRISM_FATE_DEFERRED;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) mean = mean_phase(x, n);
    __syncthreads();
    deviate(x, n, mean);
    __syncthreads();
    if (threadIdx.x == 0) stats_phase(x, n, K_rem, tau, mean, stats);
    return;
  }
  sort_phase(sc, n, reinterpret_cast<unsigned long long *>(xx), ws);
  prefix_phase(sc, n, k_req, &distinct, x, xx, P, Q, ws);
  for (int i = threadIdx.x; i <= n; i += blockDim.x) { ws.P[i] = P[i]; ws.Q[i] = Q[i]; }
}

__global__ __launch_bounds__(256) void route_table_kernel(int m, int n, const double *__restrict__ stats, RouteWs ws) {
  if (stats[2] == 0.0 || m >= ws.arg[0]) return;
  table_phase(m, n, ws, blockIdx.x * 4 + (threadIdx.x >> 6), gridDim.x * 4);
}

__global__ __launch_bounds__(1024) void route_fate_kernel(int n, int K_rem, int8_t *__restrict__ fate, double *__restrict__ stats, RouteWs ws) {
  __shared__ RouteShared sh;
  __shared__ __align__(16) double ranked[PRISM_MAX_CANDS];
  if (stats[2] == 0.0 || ws.arg[0] <= 1) return;
  for (int r = threadIdx.x; r < n; r += blockDim.x) ranked[r] = ws.ranked[r];
  fate_phase(ws.arg[0], n, K_rem, fate, stats, ranked, ws, sh);
}

static RouteWs carve(void *workspace, int n, int k) {
  RouteWs ws;
  char *p = (char *)workspace;
  const size_t dn = (size_t)round_up((n + 1) * sizeof(double), 256);
  ws.ranked = (double *)p; p += dn;
  ws.P = (double *)p; p += dn;
  ws.Q = (double *)p; p += dn;
  ws.E0 = (double *)p; p += dn;
  ws.E1 = (double *)p; p += dn;
  ws.order = (int32_t *)p; p += round_up((n + 1) * sizeof(int32_t), 256);
  ws.arg = (int32_t *)p;
  (void)k;
  return ws;
}

size_t route_workspace_bytes(int n, int k) {
  return 5 * (size_t)round_up((n + 1) * sizeof(double), 256) + (size_t)round_up((n + 1) * sizeof(int32_t), 256) +
         (size_t)round_up((size_t)(k + 1) * (n + 1) * sizeof(int32_t), 256);
}

int launch_route(const float *scores, int n, int K_rem, int n_clusters, float tau, int8_t *fate, double *stats,
                 void *workspace, hipStream_t s, const HostPost &post) {
  PRISM_REQUIRE(scores && fate && stats && workspace, PRISM_EINVAL, "route: null argument");
  PRISM_REQUIRE(n >= 1 && n <= PRISM_MAX_CANDS, PRISM_EINVAL, "route: n = %d outside 1..%d", n, PRISM_MAX_CANDS);
  PRISM_REQUIRE(n_clusters >= 2 && n_clusters <= PRISM_MAX_CLUSTERS, PRISM_EINVAL, "route: n_clusters = %d outside 2..%d",
                n_clusters, PRISM_MAX_CLUSTERS);
  PRISM_REQUIRE(K_rem >= 1 && tau >= 0.f, PRISM_EINVAL, "route: K_rem = %d, tau = %g", K_rem, (double)tau);
  if (n <= kOneGroup) {
    route_small_kernel<<<1, 512, 0, s>>>(scores, n, K_rem, n_clusters, tau, fate, stats, post);
    PRISM_HIP(hipGetLastError());
    return PRISM_OK;
  }
  const RouteWs ws = carve(workspace, n, n_clusters);
  route_prepare_kernel<<<2, 1024, 0, s>>>(scores, n, K_rem, n_clusters, tau, fate, stats, ws);
  PRISM_HIP(hipGetLastError());
  for (int m = 2; m < n_clusters; ++m) {
    route_table_kernel<<<std::min(cdiv(n, 4), 1024), 256, 0, s>>>(m, n, stats, ws);
    PRISM_HIP(hipGetLastError());
  }
  route_fate_kernel<<<1, 1024, 0, s>>>(n, K_rem, fate, stats, ws);
  PRISM_HIP(hipGetLastError());
  return post.flag ? launch_post_host(stats, post, s) : PRISM_OK;
}

// ---- the same check for callers that cannot allocate --------------------------------------------------------------
// The kernel's workspace (ranked scores, prefix sums, two cost rows, rank order, the argmin table) lives in a
// file-scope device array sized for the largest check the library accepts.  Every device that loads the library holds
// its own copy at its own address, looked up once per device.  The kernel writes every workspace entry before it reads
// it, so nothing has to be cleared between calls; calls that overlap on one device share the array and race.
static constexpr size_t up256(size_t v) { return (v + 255) / 256 * 256; }
static constexpr size_t kRouteScratchBytes =
    5 * up256((PRISM_MAX_CANDS + 1) * sizeof(double)) + up256((PRISM_MAX_CANDS + 1) * sizeof(int32_t)) +
    up256((size_t)(PRISM_MAX_CLUSTERS + 1) * (PRISM_MAX_CANDS + 1) * sizeof(int32_t));
static __device__ __align__(256) unsigned char scratch[kRouteScratchBytes];

static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (the array's name is only a host-side handle).
static int scratch_of_current_device(void **out) {
  int dev = -1;
  PRISM_HIP(hipGetDevice(&dev));
  PRISM_REQUIRE(dev >= 0 && dev < kMaxDevices, PRISM_EUNSUPPORTED, "route: device ordinal %d not supported", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    PRISM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    PRISM_REQUIRE(p, PRISM_EHIP, "route: the static workspace has no device address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return PRISM_OK;
}

}  // namespace prism

extern "C" int prism_op_route_static(const float *scores, int32_t n, int32_t K_rem, int32_t n_clusters, float tau,
                                     int8_t *fate, double *stats, void *stream) {
  using namespace prism;
  PRISM_REQUIRE(n >= 1 && n <= PRISM_MAX_CANDS, PRISM_EINVAL, "route (static workspace): n = %d outside 1..%d", n, PRISM_MAX_CANDS);
  PRISM_REQUIRE(n_clusters >= 2 && n_clusters <= PRISM_MAX_CLUSTERS, PRISM_EINVAL,
                "route (static workspace): n_clusters = %d outside 2..%d", n_clusters, PRISM_MAX_CLUSTERS);
  PRISM_REQUIRE(route_workspace_bytes(n, n_clusters) <= kRouteScratchBytes, PRISM_EINVAL,
                "route (static workspace): the check needs more than the %zu bytes of the static workspace", kRouteScratchBytes);
  void *ws = nullptr;
  PRISM_TRY(scratch_of_current_device(&ws));
  return launch_route(scores, n, K_rem, n_clusters, tau, fate, stats, ws, (hipStream_t)stream);
}
