// Monte-Carlo calibration of thresholds under digitisation (App. B): the GPU
// simulates 4+4-bit Gaussian data with a counter-based generator and
// evaluates the multi-receiver estimator on every simulated block.
#include <hip/hip_runtime.h>
#include <math.h>

#include <cmath>

#include "sk_calib.h"
#include "sk_internal.h"

namespace sk {

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Inverse CDF by table: the top bits of a 32-bit draw pick a bucket, whose
// entry holds the component at the bucket's start and the one threshold inside
// it (if any). A bucket with several thresholds is marked and its draws count
// all the thresholds; with 2^11 buckets only the tails of small RMS have such.
constexpr int MC_BUCKET_BITS = 11;
constexpr int MC_BUCKETS = 1 << MC_BUCKET_BITS;
constexpr int MC_WG = 256;
constexpr int MC_PAIRS = 512;      // (estimate, input) pairs whose sums a workgroup holds at once
constexpr int32_t MC_MANY = 1 << 20;

struct McArgs {
  uint64_t key;
  int32_t n_inputs, block_len, estimator, n_thr;
  int64_t n_sim, n_groups;
  int32_t per_group;     // estimates a workgroup takes at a time (per_group * n_inputs <= MC_PAIRS, or 1)
  int32_t seg_log;       // log2 of the lanes that share one input's samples
  int32_t seg_len;       // samples a lane draws
  uint32_t thr[16];
  double* values;   // [n_sim]
};

struct McEntry {
  uint32_t above;        // draws above this value take the next component
  int32_t component;     // at the bucket's start; MC_MANY: several thresholds inside
};

// U draws from counter z on: their powers added to s1, the squares to s2.
template <int U>
__device__ __forceinline__ void mc_draws(const McArgs& a, const McEntry* tab, int C, uint64_t& z, uint32_t& s1,
                                         uint32_t& s2) {
  uint32_t ure[U], uim[U];
  int re[U], im[U];
  int most = -C;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint64_t r = mix64(z);
    z += 0x9E3779B97F4A7C15ULL;
    ure[u] = (uint32_t)(r >> 32);
    uim[u] = (uint32_t)r;
    const McEntry x = tab[ure[u] >> (32 - MC_BUCKET_BITS)], y = tab[uim[u] >> (32 - MC_BUCKET_BITS)];
    re[u] = x.component + (ure[u] > x.above);
    im[u] = y.component + (uim[u] > y.above);
    most = most > re[u] ? most : re[u];
    most = most > im[u] ? most : im[u];
  }
  if (most >= MC_MANY) {
    asm volatile("");   // a branch, not selects on the usual path
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int x = -C, y = -C;
      for (int k = 0; k < a.n_thr; ++k) {
        x += a.thr[k] <= ure[u];
        y += a.thr[k] <= uim[u];
      }
      re[u] = x;
      im[u] = y;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t p = (uint32_t)(__mul24(re[u], re[u]) + __mul24(im[u], im[u]));
    s1 += p;
    s2 += __umul24(p, p);   // M p^2 <= 131071 * 98^2 < 2^31
  }
}

// Simulated estimates in groups of `per_group`. The lanes of a workgroup take
// (estimate, input, segment of the block) units, each walking its segment's
// draws and adding its two integer sums to the pair's in LDS, so lanes are busy
// whatever N is: one lane per input left 240 of 256 lanes idle at N = 16. Bound
// by VALU issue: a draw is two 64-bit products, the xor-shifts and two table
// reads, about 130 cycles of a SIMD per wavefront. N = 16, M = 256, 2^18
// estimates: 22.6 ms a call with one lane per input, 28 compares a draw and the
// moments on the host; 0.91 ms so (0.98 with the marked buckets looked at draw by
// draw instead of four at once).
// The FP64 sum over the inputs keeps one order: input t, t + 256, ... of each
// t < 256, then the binary tree over t.
__global__ __launch_bounds__(MC_WG) void mc_kernel(McArgs a) {
#pragma clang fp contract(off)
  __shared__ McEntry tab[MC_BUCKETS];
  __shared__ uint32_t sum1[MC_PAIRS], sum2[MC_PAIRS];
  __shared__ double acc_q[MC_PAIRS];
  __shared__ int32_t acc_n[MC_PAIRS];
  const int tid = threadIdx.x;
  const int C = a.n_thr / 2, N = a.n_inputs, M = a.block_len, E = a.per_group;
  for (int t = tid; t < MC_BUCKETS; t += MC_WG) {
    const uint32_t lo = (uint32_t)t << (32 - MC_BUCKET_BITS), hi = lo + ((1u << (32 - MC_BUCKET_BITS)) - 1);
    int below = 0, inside = 0;
    uint32_t last = 0;
    for (int k = 0; k < a.n_thr; ++k) {
      below += a.thr[k] <= lo;
      if (a.thr[k] > lo && a.thr[k] <= hi) {
        ++inside;
        last = a.thr[k];
      }
    }
    tab[t] = inside > 1 ? McEntry{~0u, MC_MANY} : McEntry{inside ? last - 1 : ~0u, below - C};
  }
  const int W = N < 256 ? N : 256;               // summing lanes per estimate
  const int slab = N < MC_PAIRS ? N : MC_PAIRS;  // inputs at a time (a multiple of 256 where N is larger)
  for (int64_t grp = blockIdx.x; grp < a.n_groups; grp += gridDim.x) {
    const int64_t e0 = grp * E;
    const int ne = a.n_sim - e0 < E ? (int)(a.n_sim - e0) : E;
    for (int k = tid; k < ne * W; k += MC_WG) {
      acc_q[k] = 0.0;
      acc_n[k] = 0;
    }
    for (int i0 = 0; i0 < N; i0 += slab) {
      const int ni = N - i0 < slab ? N - i0 : slab;
      const int pairs = ne * ni;
      for (int k = tid; k < pairs; k += MC_WG) sum1[k] = sum2[k] = 0u;
      __syncthreads();
      for (int u = tid; u < pairs << a.seg_log; u += MC_WG) {
        const int pr = u >> a.seg_log;
        const int j0 = (u & ((1 << a.seg_log) - 1)) * a.seg_len;
        const int n = M - j0 < a.seg_len ? M - j0 : a.seg_len;
        const uint64_t first = ((uint64_t)(e0 + pr / ni) * N + (i0 + pr % ni)) * (uint64_t)M + j0;
        uint64_t z = a.key + (first + 1) * 0x9E3779B97F4A7C15ULL;
        uint32_t s1 = 0, s2 = 0;
        int j = 0;
        for (; j + 4 <= n; j += 4) mc_draws<4>(a, tab, C, z, s1, s2);
        for (; j < n; ++j) mc_draws<1>(a, tab, C, z, s1, s2);
        if (n > 0) {
          atomicAdd(&sum1[pr], s1);
          atomicAdd(&sum2[pr], s2);
        }
      }
      __syncthreads();
      // Inputs t, t + 256, ... of each estimate, in order.
      for (int k = tid; k < ne * W; k += MC_WG) {
        const int e = k / W, t = k % W;
        double q = acc_q[k];
        int32_t live = acc_n[k];
        for (int i = t; i < ni; i += 256) {
          const uint32_t s1 = sum1[e * ni + i];
          if (s1 > 0) {
            const double x = (double)s1;
            q += (double)sum2[e * ni + i] / (x * x);
            live += 1;
          }
        }
        acc_q[k] = q;
        acc_n[k] = live;
      }
      __syncthreads();
    }
    for (int st = 128; st > 0; st >>= 1) {
      if (st >= W) continue;
      for (int k = tid; k < ne * st; k += MC_WG) {
        const int e = k / st, t = k % st;
        if (t + st < W) {
          acc_q[e * W + t] += acc_q[e * W + t + st];
          acc_n[e * W + t] += acc_n[e * W + t + st];
        }
      }
      __syncthreads();
    }
    for (int e = tid; e < ne; e += MC_WG) {
      const double Bq = acc_q[e * W];
      const int32_t n = acc_n[e * W];
      const double Md = (double)M, Kd = (double)n * Md;
      double V = __builtin_nan("");
      if ((int64_t)n * M >= 2 && n > 0) {
        // L = 1: A = n exactly (each S1_i / S1_i is 1).
        const double A = (double)n;
        if (a.estimator == SK_EST_TILDE)
          V = (Md + 1.0) / (Md - 1.0) * (Md * Bq / A - 1.0);
        else
          V = (Kd + 1.0) / (Kd - 1.0) * (Kd * Bq / (A * A) - 1.0);
      }
      a.values[e0 + e] = V;
    }
    __syncthreads();
  }
}

// Split of the work: enough lanes per input for about four wavefronts on every
// SIMD (2^18 lanes) while a lane keeps at least 16 draws, then the estimates
// per group that leave the fewest lanes of the last round idle.
static void mc_split(McArgs& a) {
  const int64_t N = a.n_inputs, M = a.block_len;
  int lg = 0;
  while (lg < 5 && (M >> (lg + 1)) >= 16 && a.n_sim * N < ((int64_t)1 << 18) >> lg) ++lg;
  double best = -1.0;
  for (int l = lg; l <= 5 && (l == lg || (M >> l) >= 16); ++l) {
    const int64_t len = (M + (1 << l) - 1) >> l;
    for (int64_t e = 1; e == 1 || e * N <= MC_PAIRS; ++e) {
      if (e > 1 && a.n_sim / e < 2048) break;    // several groups per CU
      const int64_t pairs = e * (N < MC_PAIRS ? N : MC_PAIRS), rounds = ((pairs << l) + MC_WG - 1) / MC_WG;
      const double eff = (double)(pairs * M) / (double)(rounds * MC_WG * len) - 0.02 * (l - lg);
      if (eff > best + 0.01) {
        best = eff;
        a.per_group = (int32_t)e;
        a.seg_log = l;
        a.seg_len = (int32_t)len;
      }
    }
  }
  a.n_groups = (a.n_sim + a.per_group - 1) / a.per_group;
}

// Moments of the valid estimates in two passes, each workgroup a strided share
// and a tree over its lanes: count and sum, then the central powers about the
// mean of all partial sums. part: [MC_PARTS][5] = count, sum, m2, m3, m4.
constexpr int MC_PARTS = 256;

template <int NV>
__device__ __forceinline__ void mc_tree(double (&v)[NV], double (*sh)[MC_WG]) {
  const int tid = threadIdx.x;
  for (int k = 0; k < NV; ++k) sh[k][tid] = v[k];
  __syncthreads();
  for (int st = MC_WG / 2; st > 0; st >>= 1) {
    if (tid < st)
      for (int k = 0; k < NV; ++k) sh[k][tid] += sh[k][tid + st];
    __syncthreads();
  }
  for (int k = 0; k < NV; ++k) v[k] = sh[k][0];
  __syncthreads();
}

__global__ __launch_bounds__(MC_WG) void mc_mean_kernel(const double* v, int64_t n, double* part) {
  __shared__ double sh[2][MC_WG];
  double t[2] = {0.0, 0.0};
  for (int64_t k = (int64_t)blockIdx.x * MC_WG + threadIdx.x; k < n; k += (int64_t)MC_PARTS * MC_WG)
    if (!isnan(v[k])) {
      t[0] += 1.0;
      t[1] += v[k];
    }
  mc_tree<2>(t, sh);
  if (threadIdx.x < 2) part[blockIdx.x * 5 + threadIdx.x] = t[threadIdx.x];
}

__global__ __launch_bounds__(MC_WG) void mc_central_kernel(const double* v, int64_t n, double* part) {
#pragma clang fp contract(off)
  __shared__ double sh[3][MC_WG];
  double m[2] = {part[threadIdx.x * 5], part[threadIdx.x * 5 + 1]};   // MC_PARTS == MC_WG
  mc_tree<2>(m, sh);
  const double mean = m[1] / m[0];
  double t[3] = {0.0, 0.0, 0.0};
  for (int64_t k = (int64_t)blockIdx.x * MC_WG + threadIdx.x; k < n; k += (int64_t)MC_PARTS * MC_WG)
    if (!isnan(v[k])) {
      const double e = v[k] - mean;
      t[0] += e * e;
      t[1] += e * e * e;
      t[2] += e * e * e * e;
    }
  mc_tree<3>(t, sh);
  if (threadIdx.x < 3) part[blockIdx.x * 5 + 2 + threadIdx.x] = t[threadIdx.x];
}

static double mc_phi(double x) { return 0.5 * erfc(-x / sqrt(2.0)); }

}  // namespace sk

extern "C" int sk_calibrate_mc(const sk_mc_desc* d, double* moments, double* d_values, void* stream) {
  using namespace sk;
  clear_error();
  if (!d || !moments || d->n_inputs < 1 || d->block_len < 2 || d->block_len > 131071 || d->clip < 1 ||
      d->clip > 7 || !(d->sigma > 0.0) || d->n_sim < 1 || d->n_sim > (1LL << 31) ||
      (d->estimator != SK_EST_HAT && d->estimator != SK_EST_TILDE)) {
    set_error("bad Monte-Carlo description");
    return SK_ERR_INVALID_ARG;
  }
  McArgs a;
  a.key = 0;
  {
    // Key = SplitMix64 output of the seed (host side, same mixing function).
    uint64_t z = d->seed;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    a.key = z ^ (z >> 31);
  }
  a.n_inputs = d->n_inputs;
  a.block_len = d->block_len;
  a.estimator = d->estimator;
  a.n_thr = 2 * d->clip;
  a.n_sim = d->n_sim;
  for (int k = 0; k < a.n_thr; ++k) {
    double s = floor(mc_phi(((double)(k - d->clip) + 0.5) / d->sigma) * 4294967296.0);
    if (s < 0) s = 0;
    if (s > 4294967295.0) s = 4294967295.0;
    a.thr[k] = (uint32_t)s;
  }
  mc_split(a);
  int dev = -1, ncu = 256;
  SK_HIP_TRY(hipGetDevice(&dev));
  (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  hipStream_t st = (hipStream_t)stream;
  // Scratch: the moments' partial sums, then the estimates if the caller does not take them.
  const size_t part_bytes = sizeof(double) * 5 * MC_PARTS;
  double* part = nullptr;
  SK_HIP_TRY(hipMalloc((void**)&part, part_bytes + (d_values ? 0 : sizeof(double) * (size_t)d->n_sim)));
  double* vals = d_values ? d_values : part + 5 * MC_PARTS;
  a.values = vals;
  // Six workgroups fit a CU (LDS).
  const int64_t grid = a.n_groups < 6 * (int64_t)ncu ? a.n_groups : 6 * (int64_t)ncu;
  mc_kernel<<<dim3((unsigned)grid), dim3(MC_WG), 0, st>>>(a);
  mc_mean_kernel<<<dim3(MC_PARTS), dim3(MC_WG), 0, st>>>(vals, d->n_sim, part);
  mc_central_kernel<<<dim3(MC_PARTS), dim3(MC_WG), 0, st>>>(vals, d->n_sim, part);
  hipError_t le = hipGetLastError();
  double h[MC_PARTS][5];
  hipError_t ce = le == hipSuccess ? hipMemcpyAsync(h, part, part_bytes, hipMemcpyDeviceToHost, st) : le;
  hipError_t se = hipStreamSynchronize(st);
  (void)hipFree(part);
  if (le != hipSuccess || ce != hipSuccess || se != hipSuccess) {
    set_error("Monte-Carlo launch failed: %s", hipGetErrorString(le != hipSuccess ? le : (ce != hipSuccess ? ce : se)));
    return SK_ERR_DEVICE;
  }
  double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int p = 0; p < MC_PARTS; ++p)
    for (int k = 0; k < 5; ++k) t[k] += h[p][k];
  const double n = t[0], pv = n > 0 ? t[2] / n : NAN;
  moments[0] = n > 0 ? t[1] / n : NAN;
  moments[1] = n > 1 ? t[2] / (n - 1) : NAN;
  moments[2] = (n > 0 && pv > 0) ? (t[3] / n) / pow(pv, 1.5) : NAN;
  moments[3] = (n > 0 && pv > 0) ? (t[4] / n) / (pv * pv) - 3.0 : NAN;
  return SK_OK;
}
