// Pass B device code shared by the single-plan and batched kernels: the
// normaliser window (Eq. discreteMean, running form), the array combine
// (Eq. normedSum1, normedSum2), the estimator (Eq. avgSK, final) and the
// flags (Sec. 3.2).
//
// Positions. Per (channel f, input i) the blocks of a call are positions
// b = 0 .. B-1; the history, the last H <= L-1 blocks of earlier calls, sits
// at positions -H .. -1. The window of block b is [max(b - L + 1, -H), b].
//
// State. The history is kept as suffix sums HS(y) = sum of S1 over positions
// [y, 0), y in [-H, 0) (HS(0) = 0, and HS(y) = HS(-H) for y < -H), one int32
// per (f, slot, i) with slot = y + L - 1. A history block is the difference
// of two neighbours, and the window's history part is one value.
//
// Kernels.
//   scan     (L >= 2; scan_chunks_body for plans, scan_body for batches, for runs
//            of blocks and for chunks of one) exclusive prefix sums of S1 at the
//            chunk boundaries of the call, PC[k] = sum of S1 over [0, k R) (mod
//            2^32: every difference that is used is a window sum < 2^31, so it is
//            exact), one lane per (f, i), a workgroup's wavefronts over consecutive
//            chunk ranges joined through LDS. It also carries the older
//            history into the next call's suffix sums when a call is shorter
//            than the window.
//   combine  one workgroup per (f, chunk k of R blocks), one wavefront per
//            64 V inputs. The window sum before the chunk is at most two
//            prefix values, R - 1 edge rows and one history value; then the
//            sliding update P += S1[b] - S1[b - L] over the chunk. Per input
//            FP64 S1/P and S2/P^2 and the raw int sums, wavefront sums in a
//            fixed tree, wavefronts joined in LDS in a fixed order, then the
//            estimator and flags of the chunk's blocks. It also writes the
//            next call's history suffix sums for its blocks.
//   step     the combine for calls with prefix sums and one group of inputs per
//            wavefront: a wavefront walks a run of up to 16 blocks (below).
// Every load of a wavefront is issued before any of them is used, so a
// combine wavefront costs one memory round trip.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sk_internal.h"
#include "sk_wave_dev.h"

namespace sk {

template <int V>
struct IVec;
template <>
struct IVec<1> {
  int32_t v[1];
  __device__ __forceinline__ void load(const int32_t* p) { v[0] = *p; }
  __device__ __forceinline__ void store(int32_t* p) const { *p = v[0]; }
};
template <>
struct IVec<4> {
  int32_t v[4];
  // Rows of any N are 4-byte aligned, which is all a 16-byte access needs.
  typedef int32_t vec __attribute__((ext_vector_type(4), aligned(4)));
  __device__ __forceinline__ void load(const int32_t* p) {
    const vec q = *reinterpret_cast<const vec*>(p);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  }
  __device__ __forceinline__ void store(int32_t* p) const {
    *reinterpret_cast<vec*>(p) = vec{v[0], v[1], v[2], v[3]};
  }
};

template <int V>
__device__ __forceinline__ void zero(IVec<V>& x) {
#pragma unroll
  for (int k = 0; k < V; ++k) x.v[k] = 0;
}

// ------------------------------------------------------------------ estimator

// Eq. originalSK: (M+1)/(M-1) (M S2 / S1^2 - 1), NaN where S1 = 0.
__device__ __forceinline__ float per_input_sk(int32_t s1, int32_t s2, int32_t block_len) {
#pragma clang fp contract(off)
  if (s1 == 0) return __builtin_nanf("");
  const double Md = (double)block_len, x = (double)s1;
  return (float)((Md + 1.0) / (Md - 1.0) * (Md * (double)s2 / (x * x) - 1.0));
}

// 1/p for p >= 1: the hardware reciprocal estimate (relative error about
// 2^-24 on gfx950) refined by two Newton steps, each squaring the error, to
// within an ulp of the correctly rounded quotient. One step would leave
// about 2^-48, enough for the tolerance on V but not for exact results such
// as V = 0 on constant-modulus input. S1/P and S2/P^2 then cost multiplies.
__device__ __forceinline__ double recip_pos(double p) {
  double r = __builtin_amdgcn_rcp(p);
  double e = __builtin_fma(-p, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-p, r, 1.0);
  return __builtin_fma(r, e, r);
}

// Estimator and flags from the combined sums (Eq. avgSK, final; Sec. 3.2).
// Contraction is off so the rounding steps are the plain ones.
__device__ __forceinline__ void finish(const PassBArgs& a, int f, int b, double A, double Bq, int64_t R1, int64_t R2,
                                       int32_t n) {
#pragma clang fp contract(off)
  const int64_t K = (int64_t)n * a.block_len;
  const double Kd = (double)K, Md = (double)a.block_len;
  bool invalid = K < 2;
  double V = 0.0;
  if (a.window == 0) {
    invalid = invalid || R1 == 0;
    if (!invalid) {
      // Eq. (2) over all K samples, numerator K R2 - R1^2 formed exactly.
      const __int128 num = (__int128)K * (__int128)R2 - (__int128)R1 * (__int128)R1;
      const __int128 den = (__int128)R1 * (__int128)R1;
      const double nd = (double)(int64_t)(num >> 64) * 18446744073709551616.0 + (double)(uint64_t)num;
      const double dd = (double)(int64_t)(den >> 64) * 18446744073709551616.0 + (double)(uint64_t)den;
      V = (Kd + 1.0) / (Kd - 1.0) * (nd / dd);
    }
  } else {
    invalid = invalid || A == 0.0;
    if (!invalid) {
      if (a.estimator == SK_EST_TILDE)
        V = (Md + 1.0) / (Md - 1.0) * (Md * Bq / (double)n - 1.0);
      else
        V = (Kd + 1.0) / (Kd - 1.0) * (Kd * Bq / (A * A) - 1.0);
    }
  }
  uint8_t fl;
  double sig = __builtin_nan("");
  if (invalid) {
    V = __builtin_nan("");
    fl = SK_FLAG_INVALID;
  } else {
    double e0 = 1.0;
    if (a.estimator == SK_EST_HAT && a.window == 1) e0 = ((Kd + 1.0) * (Md - 1.0)) / ((Kd - 1.0) * (Md + 1.0));
    const double E = e0 + a.expect_offset;
    const double s = a.sigma_override > 0.0 ? a.sigma_override : sqrt(4.0 / Kd);
    double lo = E - a.k_sigma * s, hi = E + a.k_sigma * s;
    if (a.thresholds) {
      lo = a.thresholds[2 * n];
      hi = a.thresholds[2 * n + 1];
    }
    fl = (V < lo ? SK_FLAG_LOW : 0) | (V > hi ? SK_FLAG_HIGH : 0);
    sig = (V - E) / s;
  }
  const int64_t o = (int64_t)f * a.n_blocks + b;
  if (a.significance) a.significance[o] = (float)sig;
  if (a.r1) a.r1[o] = R1;
  if (a.r2) a.r2[o] = R2;
  if (a.v) a.v[o] = (float)V;
  if (a.flags) a.flags[o] = fl;
  if (a.n_eff) a.n_eff[o] = n;
}

// Index of the calling wavefront in its workgroup, in a scalar register (the
// compiler cannot tell on its own that it is the same for every lane, and
// would keep everything derived from it per lane).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// ------------------------------------------------------------------ scan

constexpr int SCAN_MAX_WAVES = 16;

// History rows a scan wavefront moves per group (all loads, then all stores).
constexpr int SHIFT_ROWS = 16;

// History blocks that stay in the window of the next call (a call shorter
// than the window): their suffix sums grow by the whole call, `carry`.
// Next-call slot s holds position s - Hc, which is old position s - Hc + B,
// so it reads old slot s + B. Wavefront w of W takes groups of SHIFT_ROWS
// rows; a group's loads all issue before its stores (the two history buffers
// are distinct), so a short call against a long window does not walk its
// rows one load at a time.
__device__ __forceinline__ void shift_history(const PassBArgs& a, int f, int i, bool active, uint32_t carry,
                                              int w, int W) {
  const int Hc = a.hist_cap, B = a.n_blocks;
  const int from = Hc - a.hist_next_len, to = Hc - B;
  if (!active || !a.hs_next || from >= to) return;
  const int64_t rowN = a.n_inputs;
  const int32_t* src = a.hs + ((int64_t)f * Hc + B) * rowN + i;
  int32_t* dst = a.hs_next + (int64_t)f * Hc * rowN + i;
  const bool had = a.hist_len > 0;
  for (int s0 = from + w * SHIFT_ROWS; s0 < to; s0 += W * SHIFT_ROWS) {
    int32_t old[SHIFT_ROWS];
#pragma unroll
    for (int j = 0; j < SHIFT_ROWS; ++j) old[j] = (had && s0 + j < to) ? src[(int64_t)(s0 + j) * rowN] : 0;
#pragma unroll
    for (int j = 0; j < SHIFT_ROWS; ++j)
      if (s0 + j < to) dst[(int64_t)(s0 + j) * rowN] = (int32_t)((uint32_t)old[j] + carry);
  }
}

// Wavefronts the history shift of one 64-input slice can use: its rows in
// SHIFT_ROWS groups (0 when the call is at least as long as the window).
__host__ __device__ __forceinline__ int64_t shift_groups(int64_t hist_next_len, int64_t n_blocks) {
  const int64_t rows = hist_next_len - n_blocks;
  return rows > 0 ? (rows + SHIFT_ROWS - 1) / SHIFT_ROWS : 0;
}

// Whether prefix row k is read: of the stepped combine's runs (a.steps chunks each)
// only their first rows and the ones their windows start at, and the call's total;
// every row at one chunk per run.
__device__ __forceinline__ bool prefix_row_read(const PassBArgs& a, int k, int window_chunks) {
  const int m = a.steps - 1;
  return (k & m) == 0 || ((k + window_chunks) & m) == 0 || k == a.n_chunks;
}

// One workgroup of W wavefronts: channel f, slice `slice` of SCAN_INPUTS inputs, one
// input per lane. Each walker holds SCAN_ROWS units (rows of S1, or pass A's chunk
// sums) per round of SCAN_ROWS times the walkers and writes its running sum at every
// chunk end that is read; the rounds carry the running prefix. The chunk length is
// read at run time (the batched kernel's problems differ in it) and divides
// SCAN_ROWS, so the registers do not depend on it. lds: W * 64 words.
//
// Bound by its rounds' round trips: 1024 inputs, 2000 blocks, L = 1024: pass B 40.4 ->
// 27.9 us against one walker of 64 inputs and 64 rows per wavefront.
constexpr int SCAN_ROWS = 32;   // two runs of the stepped combine

// Inputs per slice: a wavefront's lanes are SCAN_PARTS walkers, each of its own rows.
// Two: twice the workgroups and half the rounds for loads of whole 128-byte lines (36.9
// us with one, 30.5 with two, 37.5 with four walkers, before the plain rounds below).
constexpr int SCAN_PARTS = 2, SCAN_INPUTS = 64 / SCAN_PARTS;

__device__ __forceinline__ void scan_body(const PassBArgs& a, int f, int slice, int w, int W, uint32_t* lds) {
  // Units: the chunk sums from pass A when the call has them (every unit
  // ends a chunk), else the rows of S1 (a chunk ends every R rows).
  const int nk = a.n_chunks, B = a.n_blocks;
  const int U = a.cs ? nk : B;
  const int R = a.cs ? 1 : a.chunk, lgR = __builtin_ctz((unsigned)R);
  const int window_chunks = a.window >> __builtin_ctz((unsigned)a.chunk);
  const int lane = threadIdx.x & (SCAN_INPUTS - 1);
  w = w * SCAN_PARTS + (int)(threadIdx.x & 63) / SCAN_INPUTS;
  W *= SCAN_PARTS;
  const int i = slice * SCAN_INPUTS + lane;
  const bool active = i < a.n_inputs;
  const int64_t rowN = a.n_inputs;
  uint32_t* pc = a.pc + (int64_t)f * (nk + 1) * rowN + i;
  if (w == 0 && active) pc[0] = 0u;
  const int32_t* src = a.cs ? a.cs + (int64_t)f * nk * rowN + i : a.s1 + (int64_t)f * B * rowN + i;
  uint32_t carry = 0;
  // Rounds wholly inside the call where only every 16th row's sum is read: no row
  // bounds and two stores a lane (bound by its instructions otherwise: 30.5 -> 21 us for
  // 71 MB of S1 in 12 problems). Offsets of 32 bits from the round's first row.
  const bool by_16 = a.chunk * a.steps == 16 && (window_chunks & (a.steps - 1)) == 0 && !a.cs &&
                     rowN <= 1 << 20;
  const uint32_t lane_off = (uint32_t)(w * SCAN_ROWS) * (uint32_t)rowN * 4u + (uint32_t)(active ? i : a.n_inputs - 1) * 4u;
  const uint8_t* chan = reinterpret_cast<const uint8_t*>(a.s1 + (int64_t)f * B * rowN);
  for (int base = 0; base < U; base += SCAN_ROWS * W) {
    const int r0 = base + w * SCAN_ROWS;
    uint32_t x[SCAN_ROWS];
    const bool plain = by_16 && base + SCAN_ROWS * W <= U;
    if (plain) {
      const uint8_t* row = chan + (int64_t)base * rowN * 4;
#pragma unroll
      for (int r = 0; r < SCAN_ROWS; ++r) {
        x[r] = *reinterpret_cast<const uint32_t*>(row + lane_off);
        row += rowN * 4;
      }
    } else {
      const int32_t* p = src + (int64_t)r0 * rowN;
#pragma unroll
      for (int r = 0; r < SCAN_ROWS; ++r) x[r] = (active && r0 + r < U) ? (uint32_t)p[(int64_t)r * rowN] : 0u;
    }
    uint32_t half = 0, tot = 0;
#pragma unroll
    for (int r = 0; r < SCAN_ROWS / 2; ++r) {
      half += x[r];
      tot += x[SCAN_ROWS / 2 + r];
    }
    tot += half;
    lds[w * SCAN_INPUTS + lane] = tot;
    __syncthreads();
    uint32_t off = carry, all = carry;
    for (int q = 0; q < W; ++q) {
      const uint32_t t = lds[q * SCAN_INPUTS + lane];
      if (q < w) off += t;
      all += t;
    }
    carry = all;
    if (active && plain) {
      pc[(int64_t)((r0 + 16) >> lgR) * rowN] = off + half;
      pc[(int64_t)((r0 + 32) >> lgR) * rowN] = off + tot;
    } else if (active) {
#pragma unroll
      for (int r = 0; r < SCAN_ROWS; ++r) {
        off += x[r];
        const int row = r0 + r;
        // Chunk c ends at unit c R + R - 1, or at U - 1 for a short last chunk.
        const int k = (row + R) >> lgR;
        if (row < U && (((row + 1) & (R - 1)) == 0 || row == U - 1) && prefix_row_read(a, k, window_chunks))
          pc[(int64_t)k * rowN] = off;
      }
    }
    __syncthreads();
  }
  shift_history(a, f, i, active, carry, w, W);
}

// Chunks a scan lane holds per round: 64 rows of S1 in flight at most.
template <int R>
constexpr int scan_chunks_per_lane() { return 64 / R; }

// The scan of plans whose combine reads every prefix row: the chunk length fixed, so no
// row asks whether it ends a chunk, and 64 inputs per slice, so half the workgroups.
// One workgroup of W wavefronts: channel f, inputs [64 slice, 64 slice + 64),
// one input per lane. Wavefront w takes chunks [k0, k0 + C) of each round of
// C W chunks (C = 64 / R); the rounds carry the running prefix. S1 of a
// chunk is the pass A chunk sum when the call has them (a.cs), else the sum
// of its R rows. lds: W * 64 words.
//
// Bound by its rounds' round trips, and past one workgroup per CU by the registers
// that hold a second one back. Against scan_body (us, scan alone): 18.9 / 37.7 (3000
// inputs, 4 channels, 1100 blocks), 15.3 / 23.9 (4096, 4, 1024), 18.2 / 22.0 (1024, 8,
// 2048), 27.6 / 32.1 (512, 8, 4096). In chunks of one block, which store every row,
// scan_body is the better while its workgroups find a CU each: pass B 37.7 / 30.8 (2
// inputs, 3000 blocks), 31.5 / 28.2 (1024, 1, 2000), but calls of 16384 inputs, 500
// blocks, L = 1000 take 120.5 / 125.7. In chunks of two, while they leave half the CUs:
// 61.8 / 57.5 (64, 4, 6000), 27.5 / 26.2 (1024, 1, 2000), but 35.7 / 36.4 (2048, 2, 1500).
template <int R>
__device__ __forceinline__ void scan_chunks_body(const PassBArgs& a, int f, int slice, int w, int W, uint32_t* lds) {
  constexpr int C = scan_chunks_per_lane<R>();
  const int lane = threadIdx.x & 63;
  const int i = slice * 64 + lane;
  const bool active = i < a.n_inputs;
  const int nk = a.n_chunks, B = a.n_blocks;
  const int64_t rowN = a.n_inputs;
  uint32_t* pc = a.pc + (int64_t)f * (nk + 1) * rowN + i;
  if (w == 0 && active) pc[0] = 0u;
  uint32_t carry = 0;   // prefix before this round, for this lane's input
  for (int base = 0; base < nk; base += C * W) {
    const int k0 = base + w * C;
    uint32_t cs[C];
    if (a.cs) {
      const int32_t* p = a.cs + ((int64_t)f * nk + k0) * rowN + i;
#pragma unroll
      for (int j = 0; j < C; ++j) cs[j] = (active && k0 + j < nk) ? (uint32_t)p[(int64_t)j * rowN] : 0u;
    } else {
      uint32_t x[C][R];
      const int32_t* p = a.s1 + ((int64_t)f * B + (int64_t)k0 * R) * rowN + i;
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int r = 0; r < R; ++r)
          x[j][r] = (active && (k0 + j) * R + r < B) ? (uint32_t)p[(int64_t)(j * R + r) * rowN] : 0u;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        uint32_t t = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) t += x[j][r];
        cs[j] = t;
      }
    }
#pragma unroll
    for (int j = 1; j < C; ++j) cs[j] += cs[j - 1];
    lds[w * 64 + lane] = cs[C - 1];
    __syncthreads();
    uint32_t off = carry, all = carry;
    for (int q = 0; q < W; ++q) {
      const uint32_t t = lds[q * 64 + lane];
      if (q < w) off += t;
      all += t;
    }
    carry = all;
    if (active) {
#pragma unroll
      for (int j = 0; j < C; ++j)
        if (k0 + j < nk) pc[(int64_t)(k0 + j + 1) * rowN] = off + cs[j];
    }
    __syncthreads();
  }
  shift_history(a, f, i, active, carry, w, W);
}

// Waves of a workgroup of scan_chunks_body for nk chunks (or groups of history rows).
__host__ __device__ __forceinline__ int scan_chunks_waves(int64_t nk) {
  return nk < SCAN_MAX_WAVES ? (nk > 0 ? (int)nk : 1) : SCAN_MAX_WAVES;
}

// Waves per slice of a scan: a power of two covering the call's
// rows in SCAN_ROWS-row lanes, at most max_waves (a power of two: the
// workgroup's wavefronts, so slices tile it).
__host__ __device__ __forceinline__ int scan_rows_waves(int64_t n_blocks, int max_waves) {
  int W = 1;
  while (W < max_waves && (int64_t)W * SCAN_PARTS * SCAN_ROWS < n_blocks) W *= 2;
  return W;
}

// Whether a call needs the prefix scan. With a window of at most one chunk
// (L <= R) no combine workgroup reads prefix sums: a window start lies in the
// chunk before, as edge rows. When the call also spans the window
// (B >= L - 1) no older history is carried either, and the combine forms the
// next history's suffix sums from the rows it reads.
__host__ __device__ __forceinline__ bool pass_b_needs_scan(int window, int chunk, int64_t n_blocks) {
  return window >= 2 && !(window <= chunk && n_blocks >= window - 1);
}

// ------------------------------------------------------------------ combine

constexpr int COMBINE_MAX_WAVES = 8;
constexpr int COMBINE_MAX_R = 4;

struct CombineShared {
  double A[COMBINE_MAX_R][COMBINE_MAX_WAVES];
  double Q[COMBINE_MAX_R][COMBINE_MAX_WAVES];
  int64_t R1[COMBINE_MAX_R][COMBINE_MAX_WAVES];
  int64_t R2[COMBINE_MAX_R][COMBINE_MAX_WAVES];
  int32_t n[COMBINE_MAX_R][COMBINE_MAX_WAVES];
};

// Element `e` of a per-channel array. OFF32: the offset is a 32-bit byte
// count added to a uniform base, so each load takes one scalar base and a
// vector offset (fewer scalar registers than a 64-bit address per row).
template <bool OFF32>
__device__ __forceinline__ const int32_t* elem_at(const int32_t* base, int64_t e) {
  if constexpr (OFF32)
    return reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(base) + (uint32_t)((uint32_t)e * 4u));
  else
    return base + e;
}

// Chunk k of channel f, wavefront w of W. R blocks per chunk, V inputs per
// lane, RI the unsigned type of a lane's R1/R2 sums, OFF32 when every
// per-channel array holds fewer than 2^30 elements.
//
// Every lane loads: a lane past the last input reads the last V inputs (in
// bounds) and contributes nothing; the lane of a last group of fewer than V
// inputs (N % V != 0) reads the last V too, counts those from its own first
// input on, and stores what its neighbour stores for the others. Loads that a chunk does not
// need are replaced by zeros in wavefront-uniform branches.
template <int V, int R, typename RI, bool OFF32>
__device__ __forceinline__ void combine_body(const PassBArgs& a, int k, int f, int w, int W, CombineShared& sh,
                                             bool live = true) {
  static_assert(R >= 1 && R <= COMBINE_MAX_R && (R & (R - 1)) == 0, "R a power of two <= 4");
  if (!live) {
    // A wavefront group with no chunk: meet the workgroup's one barrier.
    __syncthreads();
    return;
  }
  constexpr int RO = R > 1 ? R - 1 : 1;               // old-row slots
  const int lane = threadIdx.x & 63;
  const int N = a.n_inputs, L = a.window, H = a.hist_len, B = a.n_blocks;
  const int b0 = k * R;
  const int nb = B - b0 < R ? B - b0 : R;
  const int wa = b0 - L + 1;                          // first position of block b0's window
  const int n_groups = (N + 64 * V - 1) / (64 * V);
  // Prefix values the window start needs (L >= 2): PC[k] - PC[kc], kc the
  // first chunk boundary at or after max(wa, 0); positions [max(wa, 0), kc R)
  // are edge rows, a subset of the R - 1 old rows [wa, wa + R - 1).
  const int kc = wa <= 0 ? 0 : (wa + R - 1) / R;
  const bool use_pc = L >= 2 && kc < k;
  const bool scan_free = L >= 2 && !pass_b_needs_scan(L, R, B);   // no prefix sums this call
  const int edges = L >= 2 && wa > 0 ? (kc * R < b0 ? kc * R : b0) - wa : 0;
  const int hn = a.hist_next_len;
  const int tail_from = B - hn;                       // first position of the next history
  const bool tail = L >= 2 && a.hs_next && b0 + nb > tail_from;   // this chunk writes next-history sums
  const bool head = L >= 2 && wa < 0 && H > 0;        // the window reaches into the history
  const int64_t rowF = (int64_t)f * B;
  // Channel bases (uniform).
  const int32_t* s1c = a.s1 + rowF * N;
  const int32_t* s2c = a.s2 + rowF * N;
  const int32_t* pcc = reinterpret_cast<const int32_t*>(a.pc) + (int64_t)f * (a.n_chunks + 1) * N;
  const int32_t* hsc = a.hs + (int64_t)f * a.hist_cap * N;

  double accA[R], accQ[R];
  RI acc1[R], acc2[R];
  int cnt[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    accA[j] = accQ[j] = 0.0;
    acc1[j] = acc2[j] = 0;
    cnt[j] = 0;
  }

  for (int g = w; g < n_groups; g += W) {
    const int i0 = (g * 64 + lane) * V;
    const bool active = i0 < N;
    const int il = i0 < N - V ? i0 : N - V;           // the inputs this lane loads
    IVec<V> x1[R], x2[R], old[RO], hsv[R], pck, pcl, pct;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j < nb) {
        const int64_t e = (int64_t)(b0 + j) * N + il;
        x1[j].load(elem_at<OFF32>(s1c, e));
        x2[j].load(elem_at<OFF32>(s2c, e));
      } else {
        zero(x1[j]);
        zero(x2[j]);
      }
    }
    if (L >= 2) {
#pragma unroll
      for (int j = 0; j < RO; ++j) {
        const int y = wa + j;               // rows past the call's end are never used
        if (R > 1 && y >= 0 && y < B) old[j].load(elem_at<OFF32>(s1c, (int64_t)y * N + il));
        else zero(old[j]);
      }
      if (head) {
        // History suffix sums at positions wa .. wa + R - 1 (clamped to -H;
        // positions >= 0 have none). Old rows in the history are differences.
#pragma unroll
        for (int j = 0; j < R; ++j) {
          int y = wa + j;
          if (y < 0) hsv[j].load(elem_at<OFF32>(hsc, (int64_t)((y < -H ? -H : y) + a.hist_cap) * N + il));
          else zero(hsv[j]);
        }
#pragma unroll
        for (int j = 0; j < RO; ++j) {
          if (R > 1 && wa + j < 0) {
#pragma unroll
            for (int q = 0; q < V; ++q) old[j].v[q] = hsv[j].v[q] - (wa + j + 1 < 0 ? hsv[j + 1].v[q] : 0);
          }
        }
      } else {
        zero(hsv[0]);
      }
      if (!scan_free && (use_pc || tail) && k > 0) pck.load(elem_at<OFF32>(pcc, (int64_t)k * N + il));
      else zero(pck);
      if (use_pc && kc > 0) pcl.load(elem_at<OFF32>(pcc, (int64_t)kc * N + il));
      else zero(pcl);
      if (tail && !scan_free) pct.load(elem_at<OFF32>(pcc, (int64_t)a.n_chunks * N + il));
      if (tail && scan_free) {
        // S1 from the chunk's first block to the end of the call: its own rows
        // plus the at most R - 2 rows after it (pck is zero, so the next
        // history's suffix sums below come out as pct minus the rows before).
        IVec<V> after;
        zero(after);
#pragma unroll
        for (int j = 0; j < RO; ++j) {
          const int y = b0 + nb + j;
          if (R > 1 && y < B) {
            IVec<V> r;
            r.load(elem_at<OFF32>(s1c, (int64_t)y * N + il));
#pragma unroll
            for (int q = 0; q < V; ++q) after.v[q] = (int32_t)((uint32_t)after.v[q] + (uint32_t)r.v[q]);
          }
        }
#pragma unroll
        for (int q = 0; q < V; ++q) {
          uint32_t t = (uint32_t)after.v[q];
#pragma unroll
          for (int j = 0; j < R; ++j)
            if (j < nb) t += (uint32_t)x1[j].v[q];
          pct.v[q] = (int32_t)t;
        }
      }
    }
    uint32_t use = active ? (1u << V) - 1 & ~0u << (i0 - il) : 0u;
    if (a.mask) {
#pragma unroll
      for (int q = 0; q < V; ++q)
        if (a.mask[(int64_t)f * N + il + q] == 0) use &= ~(1u << q);
    }

    // Window sums, block by block (uint32 arithmetic, exact below 2^31).
    uint32_t P[V], pre[V];
    if (L >= 2) {
#pragma unroll
      for (int q = 0; q < V; ++q) {
        P[q] = (uint32_t)hsv[0].v[q] + (use_pc ? (uint32_t)pck.v[q] - (uint32_t)pcl.v[q] : 0u);
        pre[q] = (uint32_t)pck.v[q];                  // S1 of this call before the block
      }
#pragma unroll
      for (int j = 0; j < RO; ++j)
        if (j < edges) {
#pragma unroll
          for (int q = 0; q < V; ++q) P[q] += (uint32_t)old[j].v[q];
        }
    }
    uint32_t inc[R];                                  // bit q: input q of block j is included
    bool all_in = true;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      inc[j] = 0;
      if (j >= nb) break;
      if (L >= 2) {
#pragma unroll
        for (int q = 0; q < V; ++q) {
          if (j > 0) P[q] -= (uint32_t)old[j - 1].v[q];
          P[q] += (uint32_t)x1[j].v[q];
        }
        if (tail && b0 + j >= tail_from) {
          if (active) {
            IVec<V> h;
#pragma unroll
            for (int q = 0; q < V; ++q) h.v[q] = (int32_t)((uint32_t)pct.v[q] - pre[q]);
            h.store(a.hs_next + ((int64_t)f * a.hist_cap + (b0 + j - B + a.hist_cap)) * N + il);
          }
        }
#pragma unroll
        for (int q = 0; q < V; ++q) pre[q] += (uint32_t)x1[j].v[q];
      } else {
#pragma unroll
        for (int q = 0; q < V; ++q) P[q] = (uint32_t)x1[j].v[q];
      }
      if (a.sk_i && active) {
        float ski[V];
#pragma unroll
        for (int q = 0; q < V; ++q) ski[q] = per_input_sk(x1[j].v[q], x2[j].v[q], a.block_len);
        float* dst = a.sk_i + (rowF + b0 + j) * N + il;
#pragma unroll
        for (int q = 0; q < V; ++q) dst[q] = ski[q];
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const bool in = (use >> q & 1u) && (int32_t)P[q] > 0;
        const uint64_t bal = __ballot(in);
        cnt[j] += __builtin_popcountll(bal);
        all_in = all_in && bal == ~0ull;
        inc[j] |= (uint32_t)in << q;
      }
      if (L >= 1) {
        // Reciprocals now, while P holds this block's window.
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const double rp = recip_pos((double)P[q]);
          if (all_in) {
            accA[j] = __builtin_fma((double)x1[j].v[q], rp, accA[j]);
            accQ[j] = __builtin_fma((double)x2[j].v[q] * rp, rp, accQ[j]);
          } else {
            const double rs = (inc[j] >> q & 1u) ? rp : 0.0;
            accA[j] = __builtin_fma((double)x1[j].v[q], rs, accA[j]);
            accQ[j] = __builtin_fma((double)x2[j].v[q] * rs, rs, accQ[j]);
          }
        }
      }
    }
    // Raw integer sums of the included inputs.
    if (all_in) {
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int q = 0; q < V; ++q) {
          acc1[j] += (RI)x1[j].v[q];
          acc2[j] += (RI)x2[j].v[q];
        }
    } else {
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const bool in = inc[j] >> q & 1u;
          acc1[j] += in ? (RI)x1[j].v[q] : (RI)0;
          acc2[j] += in ? (RI)x2[j].v[q] : (RI)0;
        }
    }
  }

  // Wavefront sums: (A, Bq) of each block as 2R doubles, (R1, R2) as 2R ints.
  {
    constexpr int NV = 2 * R;
    double dv[NV];
    RI iv[NV];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      dv[2 * j] = accA[j];
      dv[2 * j + 1] = accQ[j];
      iv[2 * j] = acc1[j];
      iv[2 * j + 1] = acc2[j];
    }
    double dout[(NV + 3) / 4];
    uint64_t iout[(NV + 3) / 4];
    wave_sums<NV>(dv, dout);
    wave_sums_wide<NV>(iv, iout);
    const int r = lane >> 4;
    if ((lane & 15) == 0) {
#pragma unroll
      for (int q = 0; q < (NV + 3) / 4; ++q) {
        const int val = wave_value_of_row(q, r);
        if (val < NV) {
          const int j = val >> 1;
          if (val & 1) {
            sh.Q[j][w] = dout[q];
            sh.R2[j][w] = (int64_t)iout[q];
          } else {
            sh.A[j][w] = dout[q];
            sh.R1[j][w] = (int64_t)iout[q];
          }
        }
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) sh.n[j][w] = cnt[j];
    }
  }
  __syncthreads();
  if (w == 0 && lane < nb) {
    const int j = lane;
    double A = 0.0, Bq = 0.0;
    int64_t R1 = 0, R2 = 0;
    int32_t n = 0;
    for (int q = 0; q < W; ++q) {
      A += sh.A[j][q];
      Bq += sh.Q[j][q];
      R1 += sh.R1[j][q];
      R2 += sh.R2[j][q];
      n += sh.n[j][q];
    }
    finish(a, f, b0 + j, A, Bq, R1, R2, n);
  }
}

// ------------------------------------------------------------------ stepped combine
//
// The combine of long calls with a window (L >= 2; up to 2048 inputs, 4 per
// lane, or up to 64, one per lane): a wavefront walks up to STEP_BLOCKS / R chunks of R blocks one after the
// other, the next chunk's rows in flight while it works on one, and carries the
// window from block to block. Only its first chunk reads prefix sums. Against one
// chunk per wavefront: one start-up (and, batched, one problem lookup), one
// barrier and one finish per run of blocks, and loads in flight throughout (CHIME,
// M = 256: scan and combine 31.4 -> 28.4 us; 1024 inputs, 8 channels, M = 64, 1024
// blocks: 39.4 -> 34.7). Bound by the memory its 106 MB come from, at about 6 TB/s.
// Per block b the in-call window is C(b) = C(b - 1) + S1[b] - S1[b - L] (rows of
// this call only) and the normaliser P(b) = C(b) + HS(b - L + 1), so each block
// needs its two rows and either S1[b - L] or one history value.
constexpr int STEP_BLOCKS = 16;

struct StepShared {
  double A[STEP_BLOCKS][COMBINE_MAX_WAVES];
  double Q[STEP_BLOCKS][COMBINE_MAX_WAVES];
  int64_t R1[STEP_BLOCKS][COMBINE_MAX_WAVES];
  int64_t R2[STEP_BLOCKS][COMBINE_MAX_WAVES];
  int32_t n[STEP_BLOCKS][COMBINE_MAX_WAVES];
};

// Whether a call takes the stepped combine (else combine_body): it has prefix sums,
// and one group of 64 `vec` inputs per wavefront.
__host__ __device__ __forceinline__ bool steps_suit(int n_inputs, int window, int vec, int chunk, int64_t n_blocks) {
  return n_inputs <= (vec == 4 ? 2048 : 64) && pass_b_needs_scan(window, chunk, n_blocks);
}

// Chunks of R blocks a wavefront walks, `waves` being the wavefronts at one chunk
// each: 16 blocks while that leaves two wavefronts per SIMD (8192 at 4 blocks: 28.4
// us against 34.1 at one chunk each), else one chunk (4096: 25.1 against 27.1).
__host__ __device__ __forceinline__ int step_chunks(int chunk, int64_t waves) {
  return waves * chunk >= 32768 ? STEP_BLOCKS / chunk : 1;
}

// Whether a plan's call takes the stepped combine, `waves` as above: where its runs
// read only every 16th prefix row, which is what makes its scan cheap. Pass B, stepped
// against scan_chunks_body and combine_body (us): 80.6 / 108.9 (2048 inputs, 4 channels,
// 4096 blocks, L = 256) and 43.4 / 53.6 (1024, 8, 2048, 256), but 111 / 108 and 57 / 52 at
// L = 33, and 33.9 / 30.9 where no runs of 16 blocks fit (2048, 4, 1000, 256). (And where
// rows keep to no 16-byte boundary, which its fewer loads bear better: 301 / 333 (301, 8,
// 20000, 100); any_window.)
__host__ __device__ __forceinline__ bool runs_suit(int n_inputs, int window, int vec, int chunk, int64_t n_blocks,
                                                   int64_t waves, bool any_window = false) {
  const int steps = step_chunks(chunk, waves);
  return steps_suit(n_inputs, window, vec, chunk, n_blocks) && steps > 1 &&
         ((window / chunk) % steps == 0 || (any_window && vec == 4 && n_inputs % 4 != 0));
}

template <int R, int V>
struct StepRows {
  IVec<V> x1[R], x2[R], old[R];   // old: S1[b - L], or (b < L - 1) the history value of b's window
};

// Blocks [b0, b0 + R) of channel f for the V inputs from il on.
template <int R, bool OFF32, int V>
__device__ __forceinline__ void step_load(const PassBArgs& a, const int32_t* s1c, const int32_t* s2c,
                                          const int32_t* hsc, int b0, int il, StepRows<R, V>& x) {
  const int N = a.n_inputs, L = a.window, B = a.n_blocks, H = a.hist_len;
  if (b0 >= L && b0 + R <= B) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      x.x1[j].load(elem_at<OFF32>(s1c, (int64_t)(b0 + j) * N + il));
      x.x2[j].load(elem_at<OFF32>(s2c, (int64_t)(b0 + j) * N + il));
      x.old[j].load(elem_at<OFF32>(s1c, (int64_t)(b0 + j - L) * N + il));
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int b = b0 + j, y = b - L + 1;
    zero(x.x1[j]);
    zero(x.x2[j]);
    zero(x.old[j]);
    if (b < B) {
      x.x1[j].load(elem_at<OFF32>(s1c, (int64_t)b * N + il));
      x.x2[j].load(elem_at<OFF32>(s2c, (int64_t)b * N + il));
      if (y > 0) x.old[j].load(elem_at<OFF32>(s1c, (int64_t)(y - 1) * N + il));
      else if (y < 0 && H > 0) x.old[j].load(elem_at<OFF32>(hsc, (int64_t)((y < -H ? -H : y) + a.hist_cap) * N + il));
    }
  }
}

// Wavefront `w` of the W of one run: chunks [k0, k0 + steps) of channel f; its
// sums go to column `col` of sh. Contains no barrier.
template <int R, typename RI, bool OFF32, int V = 4>
__device__ __forceinline__ void step_body(const PassBArgs& a, int k0, int steps, int f, int w, int col, StepShared& sh) {
  const int lane = threadIdx.x & 63;
  const int N = a.n_inputs, L = a.window, B = a.n_blocks;
  const int i0 = (w * 64 + lane) * V;
  const bool active = i0 < N;
  const int il = i0 < N - V ? i0 : N - V;
  const int64_t rowF = (int64_t)f * B;
  const int32_t* s1c = a.s1 + rowF * N;
  const int32_t* s2c = a.s2 + rowF * N;
  const int32_t* pcc = reinterpret_cast<const int32_t*>(a.pc) + (int64_t)f * (a.n_chunks + 1) * N;
  const int32_t* hsc = a.hs + (int64_t)f * a.hist_cap * N;
  const int run0 = k0 * R;
  const int run_end = run0 + steps * R < B ? run0 + steps * R : B;
  const int tail_from = B - a.hist_next_len;
  const bool run_tail = a.hs_next && run_end > tail_from;
  StepRows<R, V> cur, next;
  step_load<R, OFF32, V>(a, s1c, s2c, hsc, run0, il, cur);
  uint32_t use = active ? (1u << V) - 1 & ~0u << (i0 - il) : 0u;
  if (a.mask) {
#pragma unroll
    for (int q = 0; q < V; ++q)
      if (a.mask[(int64_t)f * N + il + q] == 0) use &= ~(1u << q);
  }
  // In-call window of block run0 - 1: rows [max(run0 - L, 0), run0), from prefix
  // sums and the rows before the first chunk boundary at or after its start.
  uint32_t C[V], suf[V];
  {
    IVec<V> p, q0, end;
    zero(p);
    zero(q0);
    zero(end);
    const int lo = run0 - L, kc = lo <= 0 ? 0 : (lo + R - 1) / R;
    if (k0 > 0) p.load(elem_at<OFF32>(pcc, (int64_t)k0 * N + il));
    if (kc > 0) q0.load(elem_at<OFF32>(pcc, (int64_t)kc * N + il));
    if (run_tail) end.load(elem_at<OFF32>(pcc, (int64_t)a.n_chunks * N + il));
    IVec<V> edge[R > 1 ? R - 1 : 1];
#pragma unroll
    for (int j = 0; j < R - 1; ++j) {
      if (lo > 0 && lo + j < kc * R && lo + j < run0) edge[j].load(elem_at<OFF32>(s1c, (int64_t)(lo + j) * N + il));
      else zero(edge[j]);
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
      C[q] = (uint32_t)p.v[q] - (uint32_t)q0.v[q];
#pragma unroll
      for (int j = 0; j < R - 1; ++j) C[q] += (uint32_t)edge[j].v[q];
      suf[q] = (uint32_t)end.v[q] - (uint32_t)p.v[q];     // S1 from the block to the call's end
    }
  }
  for (int st = 0; st < steps; ++st) {
    const int b0 = run0 + st * R;
    if (b0 >= B) break;
    if (st + 1 < steps && b0 + R < B) step_load<R, OFF32, V>(a, s1c, s2c, hsc, b0 + R, il, next);
    const int nb = B - b0 < R ? B - b0 : R;
    const bool tail = a.hs_next && b0 + nb > tail_from;
    double accA[R], accQ[R];
    RI acc1[R], acc2[R];
    int cnt[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      accA[j] = accQ[j] = 0.0;
      acc1[j] = acc2[j] = 0;
      cnt[j] = 0;
      if (j >= nb) continue;
      const int b = b0 + j;
      const bool gone = b >= L;                       // old is the row that leaves, else a history value
      uint32_t P[V];
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const uint32_t o = (uint32_t)cur.old[j].v[q];
        C[q] += (uint32_t)cur.x1[j].v[q] - (gone ? o : 0u);
        P[q] = C[q] + (gone ? 0u : o);
      }
      if (tail && b >= tail_from && active) {
        IVec<V> h;
#pragma unroll
        for (int q = 0; q < V; ++q) h.v[q] = (int32_t)suf[q];
        h.store(a.hs_next + ((int64_t)f * a.hist_cap + (b - B + a.hist_cap)) * N + il);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) suf[q] -= (uint32_t)cur.x1[j].v[q];
      if (a.sk_i && active) {
        float* dst = a.sk_i + (rowF + b) * N + il;
#pragma unroll
        for (int q = 0; q < V; ++q) dst[q] = per_input_sk(cur.x1[j].v[q], cur.x2[j].v[q], a.block_len);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const bool in = (use >> q & 1u) && (int32_t)P[q] > 0;
        cnt[j] += __builtin_popcountll(__ballot(in));
        const double rp = in ? recip_pos((double)P[q]) : 0.0;
        accA[j] = __builtin_fma((double)cur.x1[j].v[q], rp, accA[j]);
        accQ[j] = __builtin_fma((double)cur.x2[j].v[q] * rp, rp, accQ[j]);
        acc1[j] += in ? (RI)cur.x1[j].v[q] : (RI)0;
        acc2[j] += in ? (RI)cur.x2[j].v[q] : (RI)0;
      }
    }
    constexpr int NV = 2 * R;
    double dv[NV];
    RI iv[NV];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      dv[2 * j] = accA[j];
      dv[2 * j + 1] = accQ[j];
      iv[2 * j] = acc1[j];
      iv[2 * j + 1] = acc2[j];
    }
    double dout[(NV + 3) / 4];
    uint64_t iout[(NV + 3) / 4];
    wave_sums<NV>(dv, dout);
    wave_sums_wide<NV>(iv, iout);
    if ((lane & 15) == 0) {
#pragma unroll
      for (int q = 0; q < (NV + 3) / 4; ++q) {
        const int val = wave_value_of_row(q, lane >> 4);
        if (val < NV) {
          const int j = st * R + (val >> 1);
          if (val & 1) {
            sh.Q[j][col] = dout[q];
            sh.R2[j][col] = (int64_t)iout[q];
          } else {
            sh.A[j][col] = dout[q];
            sh.R1[j][col] = (int64_t)iout[q];
          }
        }
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) sh.n[st * R + j][col] = cnt[j];
    }
    cur = next;
  }
}

// Block j of a run whose W wavefronts hold columns col0 .. of sh: their sums in
// order, then the estimator and flags.
__device__ __forceinline__ void step_finish(const PassBArgs& a, int f, int b, int j, int col0, int W, const StepShared& sh) {
  double A = 0.0, Bq = 0.0;
  int64_t R1 = 0, R2 = 0;
  int32_t n = 0;
  for (int q = col0; q < col0 + W; ++q) {
    A += sh.A[j][q];
    Bq += sh.Q[j][q];
    R1 += sh.R1[j][q];
    R2 += sh.R2[j][q];
    n += sh.n[j][q];
  }
  finish(a, f, b, A, Bq, R1, R2, n);
}

// Waves of a combine workgroup for N inputs at V per lane.
__host__ __device__ __forceinline__ int combine_waves(int n_inputs, int vec) {
  const int g = (n_inputs + 64 * vec - 1) / (64 * vec);
  return g < COMBINE_MAX_WAVES ? g : COMBINE_MAX_WAVES;
}

// Whether every per-channel array of a call (S1, S2, prefix sums, history)
// holds fewer than 2^30 elements, so 32-bit byte offsets reach all of it.
__host__ __device__ __forceinline__ bool combine_offsets_fit_32(int n_inputs, int64_t n_blocks, int n_chunks,
                                                                int hist_cap) {
  const int64_t lim = (int64_t)1 << 30;
  return n_blocks * n_inputs < lim && ((int64_t)n_chunks + 1) * n_inputs < lim && (int64_t)hist_cap * n_inputs < lim;
}

// Integer type of a lane's R1/R2 sums: 32 bits while half a wavefront's S2 sums
// fit (32 V M 2^14 < 2^32, S2 of one input <= M 2^14; the last addition of the
// wavefront sum is in 64 bits), over all the groups a wavefront takes: M < 2048
// up to 2048 inputs.
__host__ __device__ __forceinline__ bool combine_sums_fit_32(int n_inputs, int vec, int block_len) {
  const int W = combine_waves(n_inputs, vec);
  const int64_t groups = (n_inputs + 64 * vec - 1) / (64 * vec);
  const int64_t per_wave = (groups + W - 1) / W;
  return per_wave * 32 * vec * (int64_t)block_len * 16384 < ((int64_t)1 << 32);
}

}  // namespace sk
