// Pass B: normaliser window, array combine, estimator and flags
// (Eq. discreteMean, normedSum1, normedSum2, avgSK, final; Sec. 3.2).
//
// The normaliser of block b is the window sum P = sum of S1 over b - L + 1 .. b
// (Eq. discreteMean is L = 1: the block's own power). Its common factor (M
// times the number of blocks in the window) is the same for every input of a
// (channel, block) and cancels in the estimator, so the weights are 1/P_i
// (Eq. normedSum1, normedSum2). Calls whose windows cost few rows take the
// window kernel below; the others the kernels of sk_pass_b_dev.h: a prefix scan
// of S1 over chunk boundaries (L >= 2), then one combine workgroup per (channel,
// chunk) that finishes its blocks.
// Every sum runs in a fixed order (lane-sequential, the fixed wavefront tree,
// wavefronts in order), so results are identical from call to call and do not
// depend on the chunk length.
#include <hip/hip_runtime.h>
#include <math.h>

#include "sk_internal.h"
#include "sk_pass_b_dev.h"

namespace sk {

__global__ __launch_bounds__(64 * SCAN_MAX_WAVES) void scan_kernel(PassBArgs a) {
  __shared__ uint32_t lds[SCAN_MAX_WAVES * 64];
  scan_body(a, blockIdx.y, blockIdx.x, wave_id(), blockDim.x >> 6, lds);
}

template <int R>
__global__ __launch_bounds__(64 * SCAN_MAX_WAVES) void scan_chunks_kernel(PassBArgs a) {
  __shared__ uint32_t lds[SCAN_MAX_WAVES * 64];
  scan_chunks_body<R>(a, blockIdx.y, blockIdx.x, wave_id(), blockDim.x >> 6, lds);
}

template <int V, int R, typename RI, bool OFF32>
__global__ __launch_bounds__(64 * COMBINE_MAX_WAVES) void combine_kernel(PassBArgs a) {
  __shared__ CombineShared sh;
  combine_body<V, R, RI, OFF32>(a, blockIdx.x, blockIdx.y, wave_id(), blockDim.x >> 6, sh);
}

// One run of a.steps chunks per workgroup.
template <int R, typename RI, bool OFF32, int V>
__global__ __launch_bounds__(64 * COMBINE_MAX_WAVES) void step_kernel(PassBArgs a) {
  __shared__ StepShared sh;
  const int steps = a.steps, f = blockIdx.y, k0 = (int)blockIdx.x * steps, W = blockDim.x >> 6;
  step_body<R, RI, OFF32, V>(a, k0, steps, f, wave_id(), wave_id(), sh);
  __syncthreads();
  const int j = threadIdx.x, b = k0 * R + j;
  if (j < steps * R && b < a.n_blocks) step_finish(a, f, b, j, 0, W, sh);
}

template <int R, bool OFF32, int V>
static void launch_step_r(const PassBArgs& a, bool fit32, dim3 grid, dim3 wg, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1) {
  if (fit32) launch_kernel(step_kernel<R, uint32_t, OFF32, V>, grid, wg, 0, s, e0, e1, a);
  else launch_kernel(step_kernel<R, uint64_t, OFF32, V>, grid, wg, 0, s, e0, e1, a);
}

template <int R>
static int launch_step(const PassBArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const bool fit32 = combine_sums_fit_32(a.n_inputs, a.vec, a.block_len);
  const bool off32 = combine_offsets_fit_32(a.n_inputs, a.n_blocks, a.n_chunks, a.hist_cap);
  const int W = combine_waves(a.n_inputs, a.vec);
  const dim3 grid((a.n_chunks + a.steps - 1) / a.steps, a.n_channels), wg(64 * W);
  if (a.vec == 1) launch_step_r<R, false, 1>(a, fit32, grid, wg, s, e0, e1);
  else if (off32) launch_step_r<R, true, 4>(a, fit32, grid, wg, s, e0, e1);
  else launch_step_r<R, false, 4>(a, fit32, grid, wg, s, e0, e1);
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

template <int V, int R>
static void launch_combine_r(const PassBArgs& a, bool fit32, dim3 grid, dim3 wg, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1) {
  const bool off32 = combine_offsets_fit_32(a.n_inputs, a.n_blocks, a.n_chunks, a.hist_cap);
  if (fit32 && off32) launch_kernel(combine_kernel<V, R, uint32_t, true>, grid, wg, 0, s, e0, e1, a);
  else if (fit32) launch_kernel(combine_kernel<V, R, uint32_t, false>, grid, wg, 0, s, e0, e1, a);
  else if (off32) launch_kernel(combine_kernel<V, R, uint64_t, true>, grid, wg, 0, s, e0, e1, a);
  else launch_kernel(combine_kernel<V, R, uint64_t, false>, grid, wg, 0, s, e0, e1, a);
}

template <int V>
static int launch_combine_v(const PassBArgs& a, bool fit32, dim3 grid, dim3 wg, hipStream_t s, hipEvent_t e0,
                            hipEvent_t e1) {
  switch (a.chunk) {
    case 1: launch_combine_r<V, 1>(a, fit32, grid, wg, s, e0, e1); break;
    case 2: launch_combine_r<V, 2>(a, fit32, grid, wg, s, e0, e1); break;
    case 4: launch_combine_r<V, 4>(a, fit32, grid, wg, s, e0, e1); break;
    default:
      set_error("pass B: chunk length %d is not 1, 2 or 4", a.chunk);
      return SK_ERR_INVALID_ARG;
  }
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

// Wavefronts of a window workgroup: 16 read no fewer rows for the call's time
// (frame256: 8.4 against 6.4 us) and spill at four blocks each.
constexpr int WINDOW_WAVES = 8;

// Window kernel: pass B in one launch, without prefix sums. A workgroup takes
// one slice of 64 V inputs of a channel (V = 1: one slice, up to 64 inputs) and X = NW R consecutive blocks, R per
// wavefront. The window sum before its first block comes from the rows
// themselves: the wavefronts share them, and each then starts from that sum, the
// blocks of the wavefronts before it and the rows those let go, all met in LDS.
// (The rows are read again by every workgroup of the slice, from L2: workgroups
// of a slice are a multiple of 8 apart where the slices are, so on one XCD.)
//
// A slice's sums of a block are the combine's wavefront sums, in the combine's
// order, so results are the same bit for bit. Up to 256 inputs they are the
// block's; above, slices meet in device memory and the last to finish a segment
// adds them in slice order and finishes its blocks. Those words are written and
// read with agent-scope atomics (past the XCDs' caches), and the count is added
// to once they have arrived, so no cache is written back. The counts start at zero:
// the call's pass A clears them.
//
// Further workgroups carry the older history on when the call is shorter than
// the window, as the scan does.
template <int R, typename RI, int V>
__global__ __launch_bounds__(64 * WINDOW_WAVES) void window_kernel(PassBArgs a, int W, int segs, int shift_wgs) {
  constexpr int NW = WINDOW_WAVES, C = 64 * V, X = NW * R, BATCH = 8;
  static_assert(X <= 64, "one wavefront finishes a segment");
  __shared__ int32_t sh_base[NW][C], sh_delta[NW][C], sh_own[NW][C], sh_after[NW][C];
  __shared__ double fin_A[X], fin_Q[X];
  __shared__ int64_t fin_R1[X], fin_R2[X];
  __shared__ int32_t fin_n[X];
  const int w = wave_id(), lane = threadIdx.x & 63;
  const int N = a.n_inputs, L = a.window, H = a.hist_len, B = a.n_blocks, Hc = a.hist_cap;
  const int n_groups = (N + C - 1) / C;
  const int hn = a.hist_next_len;
  // Rows r, r + NW, ... < end of one channel, summed for this lane's inputs.
  const auto sum_rows_of = [&](const int32_t* rows, int r, int end, int il, IVec<V>& t) {
    for (; r < end; r += BATCH * NW) {
      IVec<V> x[BATCH];
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int y = r + k * NW < end ? r + k * NW : r;
        x[k].load(rows + (int64_t)y * N + il);
      }
#pragma unroll
      for (int k = 0; k < BATCH; ++k)
        if (r + k * NW < end)
#pragma unroll
          for (int q = 0; q < V; ++q) t.v[q] = (int32_t)((uint32_t)t.v[q] + (uint32_t)x[k].v[q]);
    }
  };
  const int pairs = a.n_channels * W;
  if ((int)blockIdx.x >= pairs * segs) {
    // Older history: NW * BATCH rows of one group of inputs.
    const int t = (int)blockIdx.x - pairs * segs;
    const int fg = t / shift_wgs, f = fg / n_groups, g = fg % n_groups;
    const int i0 = (g * 64 + lane) * V, il = i0 < N - V ? i0 : N - V;
    const int from = Hc - hn, to = Hc - B;
    const int s0 = from + ((t % shift_wgs) * NW + w) * BATCH;
    const int32_t* src = a.hs + ((int64_t)f * Hc + B) * N + il;
    int32_t* dst = a.hs_next + (int64_t)f * Hc * N + il;
    IVec<V> old[BATCH], mine;
    zero(mine);
#pragma unroll
    for (int k = 0; k < BATCH; ++k)
      if (s0 + k < to) old[k].load(src + (int64_t)(s0 + k) * N);
    sum_rows_of(a.s1 + (int64_t)f * B * N, w, B, il, mine);
    mine.store(&sh_base[w][lane * V]);
    __syncthreads();
    IVec<V> all;
    zero(all);
    for (int j = 0; j < NW; ++j) {
      IVec<V> x;
      x.load(&sh_base[j][lane * V]);
#pragma unroll
      for (int q = 0; q < V; ++q) all.v[q] = (int32_t)((uint32_t)all.v[q] + (uint32_t)x.v[q]);
    }
    if (i0 < N)
#pragma unroll
      for (int k = 0; k < BATCH; ++k)
        if (s0 + k < to) {
#pragma unroll
          for (int q = 0; q < V; ++q) old[k].v[q] = (int32_t)((uint32_t)old[k].v[q] + (uint32_t)all.v[q]);
          old[k].store(dst + (int64_t)(s0 + k) * N);
        }
    return;
  }
  const int pair = (int)blockIdx.x % pairs, seg = (int)blockIdx.x / pairs;
  const int f = pair / W, slice = pair % W;
  const int b0 = seg * X, b_end = b0 + X < B ? b0 + X : B;
  const int bw = b0 + w * R;                          // this wavefront's first block
  const int nb = B - bw < 0 ? 0 : (B - bw < R ? B - bw : R);
  const int wa = bw - L + 1;                          // first position of its window
  const int lo = b0 - L + 1 > 0 ? b0 - L + 1 : 0;
  const int tail_from = B - hn;
  const bool tail = a.hs_next && b_end > tail_from;   // the segment writes next-history sums
  const int64_t rowF = (int64_t)f * B;
  const int32_t* s1c = a.s1 + rowF * N;
  const int32_t* s2c = a.s2 + rowF * N;
  const int32_t* hsc = a.hs + (int64_t)f * Hc * N;

  double accA[R], accQ[R];
  RI acc1[R], acc2[R];
  int cnt[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    accA[j] = accQ[j] = 0.0;
    acc1[j] = acc2[j] = 0;
    cnt[j] = 0;
  }
  for (int g = slice; g < n_groups; g += W) {
    const int i0 = (g * 64 + lane) * V;
    const bool active = i0 < N;
    const int il = i0 < N - V ? i0 : N - V;
    IVec<V> x1[R], x2[R], old[R], hsv[R], base, after;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j < nb) {
        x1[j].load(s1c + (int64_t)(bw + j) * N + il);
        x2[j].load(s2c + (int64_t)(bw + j) * N + il);
      } else {
        zero(x1[j]);
        zero(x2[j]);
      }
      const int y = wa + j;                           // the row that block bw + j is the last to use
      if (y >= 0 && y < B) old[j].load(s1c + (int64_t)y * N + il);
      else zero(old[j]);
      if (y < 0 && H > 0 && nb > 0) hsv[j].load(hsc + (int64_t)((y < -H ? -H : y) + Hc) * N + il);
      else zero(hsv[j]);
    }
    zero(base);
    zero(after);
    sum_rows_of(s1c, lo + w, b0, il, base);
    if (tail) sum_rows_of(s1c, b_end + w, B, il, after);
    base.store(&sh_base[w][lane * V]);
    {
      IVec<V> d, o;
#pragma unroll
      for (int q = 0; q < V; ++q) {
        uint32_t own = 0, gone = 0;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          own += (uint32_t)x1[j].v[q];
          gone += (uint32_t)old[j].v[q];
        }
        o.v[q] = (int32_t)own;
        d.v[q] = (int32_t)(own - gone);
      }
      d.store(&sh_delta[w][lane * V]);
      if (tail) {
        o.store(&sh_own[w][lane * V]);
        after.store(&sh_after[w][lane * V]);
      }
    }
    __syncthreads();
    uint32_t win[V], suf[V];                          // in-call window before the block; S1 from it to the end
#pragma unroll
    for (int q = 0; q < V; ++q) win[q] = suf[q] = 0u;
    for (int j = 0; j < NW; ++j) {
      IVec<V> x;
      x.load(&sh_base[j][lane * V]);
#pragma unroll
      for (int q = 0; q < V; ++q) win[q] += (uint32_t)x.v[q];
    }
#pragma unroll 4
    for (int j = 0; j < w; ++j) {
      IVec<V> x;
      x.load(&sh_delta[j][lane * V]);
#pragma unroll
      for (int q = 0; q < V; ++q) win[q] += (uint32_t)x.v[q];
    }
    if (tail) {
      for (int j = 0; j < NW; ++j) {
        IVec<V> x;
        x.load(&sh_after[j][lane * V]);
#pragma unroll
        for (int q = 0; q < V; ++q) suf[q] += (uint32_t)x.v[q];
      }
#pragma unroll 4
      for (int j = w; j < NW; ++j) {
        IVec<V> x;
        x.load(&sh_own[j][lane * V]);
#pragma unroll
        for (int q = 0; q < V; ++q) suf[q] += (uint32_t)x.v[q];
      }
    }
    uint32_t use = active ? (1u << V) - 1 & ~0u << (i0 - il) : 0u;
    if (a.mask) {
#pragma unroll
      for (int q = 0; q < V; ++q)
        if (a.mask[(int64_t)f * N + il + q] == 0) use &= ~(1u << q);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j >= nb) break;
      uint32_t P[V];
#pragma unroll
      for (int q = 0; q < V; ++q) {
        win[q] += (uint32_t)x1[j].v[q];
        if (j > 0) win[q] -= (uint32_t)old[j - 1].v[q];
        P[q] = win[q] + (uint32_t)hsv[j].v[q];
      }
      if (tail && bw + j >= tail_from && active) {
        IVec<V> h;
#pragma unroll
        for (int q = 0; q < V; ++q) h.v[q] = (int32_t)suf[q];
        h.store(a.hs_next + ((int64_t)f * Hc + (bw + j - B + Hc)) * N + il);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) suf[q] -= (uint32_t)x1[j].v[q];
      if (a.sk_i && active) {
        float* dst = a.sk_i + (rowF + bw + j) * N + il;
#pragma unroll
        for (int q = 0; q < V; ++q) dst[q] = per_input_sk(x1[j].v[q], x2[j].v[q], a.block_len);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const bool in = (use >> q & 1u) && (int32_t)P[q] > 0;
        cnt[j] += __builtin_popcountll(__ballot(in));
        const double rp = in ? recip_pos((double)P[q]) : 0.0;
        accA[j] = __builtin_fma((double)x1[j].v[q], rp, accA[j]);
        accQ[j] = __builtin_fma((double)x2[j].v[q] * rp, rp, accQ[j]);
        acc1[j] += in ? (RI)x1[j].v[q] : (RI)0;
        acc2[j] += in ? (RI)x2[j].v[q] : (RI)0;
      }
    }
    if (g + W < n_groups) __syncthreads();            // the next group reuses the LDS rows
  }
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
    if ((lane & 15) == 0) {
#pragma unroll
      for (int q = 0; q < (NV + 3) / 4; ++q) {
        const int val = wave_value_of_row(q, lane >> 4);
        if (val < NV) {
          const int k = w * R + (val >> 1);
          if (val & 1) {
            fin_Q[k] = dout[q];
            fin_R2[k] = (int64_t)iout[q];
          } else {
            fin_A[k] = dout[q];
            fin_R1[k] = (int64_t)iout[q];
          }
        }
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) fin_n[w * R + j] = cnt[j];
    }
  }
  __syncthreads();
  if (w != 0) return;
  const bool mine = b0 + lane < b_end;
  if (W == 1) {
    if (mine) finish(a, f, b0 + lane, fin_A[lane], fin_Q[lane], fin_R1[lane], fin_R2[lane], fin_n[lane]);
    return;
  }
  const int64_t plane = (int64_t)a.n_channels * B * W;
  uint64_t* part = reinterpret_cast<uint64_t*>(a.part) + (rowF + b0 + lane) * W;
  const auto put = [&](int k, uint64_t v) {
    __hip_atomic_store(part + k * plane + slice, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const auto get = [&](int k, int q) {
    return __hip_atomic_load(part + k * plane + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (mine) {
    put(0, __builtin_bit_cast(uint64_t, fin_A[lane]));
    put(1, __builtin_bit_cast(uint64_t, fin_Q[lane]));
    put(2, (uint64_t)fin_R1[lane]);
    put(3, (uint64_t)fin_R2[lane]);
    put(4, (uint64_t)fin_n[lane]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // the words have arrived
  uint32_t* done = a.done + f * segs + seg;
  uint32_t before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  before = __builtin_amdgcn_readfirstlane(before);
  if (before != (uint32_t)W - 1) return;
  asm volatile("" ::: "memory");
  if (mine) {
    uint64_t v[COMBINE_MAX_WAVES][5];
#pragma unroll
    for (int q = 0; q < COMBINE_MAX_WAVES; ++q)
#pragma unroll
      for (int k = 0; k < 5; ++k) v[q][k] = get(k, q < W ? q : 0);   // no branch, so all are in flight together (7.8 -> 6.8 us, 1000 inputs)
    double A = 0.0, Bq = 0.0;
    int64_t R1 = 0, R2 = 0;
    int32_t n = 0;
#pragma unroll
    for (int q = 0; q < COMBINE_MAX_WAVES; ++q) {
      if (q >= W) break;
      A += __builtin_bit_cast(double, v[q][0]);
      Bq += __builtin_bit_cast(double, v[q][1]);
      R1 += (int64_t)v[q][2];
      R2 += (int64_t)v[q][3];
      n += (int32_t)v[q][4];
    }
    finish(a, f, b0 + lane, A, Bq, R1, R2, n);
  }
}

// Workgroups per channel and group of inputs that move the older history rows that stay.
static int window_shift_wgs(const PassBArgs& a) {
  const int rows = a.hist_next_len - a.n_blocks;
  return a.hs_next && rows > 0 ? (rows + WINDOW_WAVES * 8 - 1) / (WINDOW_WAVES * 8) : 0;
}

// (A launch holds fewer than 2^32 lanes, 2^23 workgroups; those of the blocks are below
// 2^18. The scan walks such a history in loops.)
bool pass_b_window_fits(const PassBArgs& a) {
  const int64_t groups = (a.n_inputs + 64 * a.vec - 1) / (64 * a.vec);
  return a.n_channels * groups * window_shift_wgs(a) < 1 << 22;
}

template <int R, int V>
static int launch_window(const PassBArgs& a, hipStream_t s, PassEvents ev) {
  constexpr int X = WINDOW_WAVES * R;
  const int W = combine_waves(a.n_inputs, V), segs = (a.n_blocks + X - 1) / X;
  const int shift_wgs = window_shift_wgs(a);
  const int groups = (a.n_inputs + 64 * V - 1) / (64 * V);
  const dim3 grid(a.n_channels * (W * segs + groups * shift_wgs)), wg(64 * WINDOW_WAVES);
  if (combine_sums_fit_32(a.n_inputs, V, a.block_len))
    launch_kernel(window_kernel<R, uint32_t, V>, grid, wg, 0, s, ev.start, ev.stop, a, W, segs, shift_wgs);
  else
    launch_kernel(window_kernel<R, uint64_t, V>, grid, wg, 0, s, ev.start, ev.stop, a, W, segs, shift_wgs);
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

int launch_pass_b(const PassBArgs& args, hipStream_t s, PassEvents ev) {
  PassBArgs a = args;
  if (a.n_blocks <= 0) return SK_OK;
  if (a.direct) {
    switch (a.chunk) {
      case 1: return a.vec == 4 ? launch_window<1, 4>(a, s, ev) : launch_window<1, 1>(a, s, ev);
      case 2: return a.vec == 4 ? launch_window<2, 4>(a, s, ev) : launch_window<2, 1>(a, s, ev);
      case 4: return a.vec == 4 ? launch_window<4, 4>(a, s, ev) : launch_window<4, 1>(a, s, ev);
    }
    set_error("pass B: chunk length %d is not 1, 2 or 4", a.chunk);
    return SK_ERR_INVALID_ARG;
  }
  const int F = a.n_channels;
  hipEvent_t start = ev.start;
  const int64_t waves = (int64_t)a.n_chunks * F * combine_waves(a.n_inputs, 4);
  // Runs of blocks with every prefix row written, too, where a wavefront has few inputs
  // (us, against the plain combine): 75.0 / 82.2 (64 inputs, 8 channels, 8192 blocks, L =
  // 33), 56.4 / 57.7 (64, 1, 8192), but 86.9 / 84.3 (256, 8, 8192).
  const bool runs = runs_suit(a.n_inputs, a.window, a.vec, a.chunk, a.n_blocks, waves, true);
  const bool stepped = runs || (a.n_inputs <= 64 && steps_suit(a.n_inputs, a.window, a.vec, a.chunk, a.n_blocks) &&
                                step_chunks(a.chunk, waves) > 1);
  if (stepped) a.steps = step_chunks(a.chunk, waves);
  if (pass_b_needs_scan(a.window, a.chunk, a.n_blocks)) {
    // Enough wavefronts for the chunks, or for the history rows a call
    // shorter than the window moves.
    const int64_t sg = shift_groups(a.hist_next_len, a.n_blocks);
    const dim3 grid((a.n_inputs + SCAN_INPUTS - 1) / SCAN_INPUTS, F);
    if (runs || (int64_t)grid.x * F <= (a.chunk == 1 ? 256 : a.chunk == 2 ? 128 : 0)) {
      int W = scan_rows_waves(a.cs ? a.n_chunks : a.n_blocks, SCAN_MAX_WAVES);
      while (W < SCAN_MAX_WAVES && W * SCAN_PARTS < sg) W *= 2;
      const dim3 wg(64 * W);
      launch_kernel(scan_kernel, grid, wg, 0, s, start, nullptr, a);
    } else {
      const dim3 half((a.n_inputs + 63) / 64, F), wg(64 * scan_chunks_waves(sg > a.n_chunks ? sg : a.n_chunks));
      switch (a.chunk) {
        case 1: launch_kernel(scan_chunks_kernel<1>, half, wg, 0, s, start, nullptr, a); break;
        case 2: launch_kernel(scan_chunks_kernel<2>, half, wg, 0, s, start, nullptr, a); break;
        case 4: launch_kernel(scan_chunks_kernel<4>, half, wg, 0, s, start, nullptr, a); break;
        default:
          set_error("pass B: chunk length %d is not 1, 2 or 4", a.chunk);
          return SK_ERR_INVALID_ARG;
      }
    }
    SK_HIP_TRY(hipGetLastError());
    start = nullptr;
  }
  if (stepped) {
    switch (a.chunk) {
      case 1: return launch_step<1>(a, s, start, ev.stop);
      case 2: return launch_step<2>(a, s, start, ev.stop);
      case 4: return launch_step<4>(a, s, start, ev.stop);
    }
  }
  const dim3 grid(a.n_chunks, F), wg(64 * combine_waves(a.n_inputs, a.vec));
  const bool fit32 = combine_sums_fit_32(a.n_inputs, a.vec, a.block_len);
  if (a.vec == 4) return launch_combine_v<4>(a, fit32, grid, wg, s, start, ev.stop);
  return launch_combine_v<1>(a, fit32, grid, wg, s, start, ev.stop);
}

// Four inputs per lane, or one where a wavefront holds them all and rows keep to no
// 16-byte boundary: its lanes then share the work (8 channels, 20000 blocks, us, four /
// one: 53 / 40 with 5 to 63 inputs, but 53 / 69 with 65, which take two wavefronts).
int pass_b_vec(int32_t n_inputs) { return n_inputs % 4 == 0 || n_inputs > 64 ? 4 : 1; }

// Window workgroups of a call at R blocks per wavefront.
static int64_t window_workgroups(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int chunk) {
  return (int64_t)n_channels * combine_waves(n_inputs, 4) * ((n_blocks + WINDOW_WAVES * chunk - 1) / (WINDOW_WAVES * chunk));
}

int pass_b_scan_free_chunk(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int32_t window) {
  // (Input counts past 256 that are no multiple of 4 count their wavefronts by one input
  // a lane.)
  const int R = pass_b_chunk(n_inputs, n_channels, n_blocks, n_inputs % 4 && n_inputs > 256 ? 1 : pass_b_vec(n_inputs));
  return window >= 2 && !pass_b_needs_scan(window, R, n_blocks) ? R : 0;
}

// The window kernel reads up to min(L - 1, B) rows again per workgroup (and per
// 2048 inputs), the scan and the combine a bounded number per block: the line is
// at 2^17 such rows, about half a megabyte a CU, and at twice that where no
// slices have to meet. Pass B alone, window kernel against scan and combine (us):
// 6.4 / 16.8 (256 inputs, 4 channels, 192 blocks, L = 256), 9.4 / 16.4 (256, 8,
// 512, 256), 13.3 / 21 (2048, 4, 192, 256), 12.4 / 19 (2048, 4, 256, 64), 16.8 /
// 20.2 (1024, 4, 512, 512: just below), 15.3 / 18.3 (256, 4, 1024, 1024); above it
// 26.8 / 24.6 (2048, 2, 512, 1024), 25.8 / 25.6 (512, 8, 1024, 512), 41.6 / 31.4
// (2048, 4, 1024, 256).
//
// Not where the combine needs no prefix sums: one launch too, and no row again: 29.4 /
// 18.9 (2048, 4, 1024, 2), 115 / 63 (2048, 4, 4096, 4), 22 / 17 (64, 8, 4096, 2), equal at
// 12.4 / 12.6 (256, 8, 2048, 4). And not where many blocks make the slices' meeting cost
// more than a scan: from 2^16 wavefront sums of 4 slices or more on (121 / 111: 2048, 4,
// 4096, 8; 57.8 / 55.2: 1024, 8, 2048, 12; below it 30.3 / 39.2: 2048, 2, 2048, 8, with two
// slices 57.5 / 65.7: 512, 8, 4096, 12), and where the stepped combine runs, from 2^15 of
// 4 slices (32.5 / 27.4: 2048, 4, 1024, 16) or 2^16 (57.6 / 54.0: 512, 8, 4096, 16; below
// it 30.1 / 31.3: 512, 8, 2048, 16). Where the scan is one round or little more, a window
// past 16 blocks costs more than it from 7 2^12 sums on (33.3 / 29.0: 2048, 4, 1000, 33;
// 60.5 / 50.0: 3000, 4, 1100, 32; below it 18.0 / 24.2: 2048, 2, 1024, 64). Where 4 does
// not divide the inputs, rows off 16-byte boundaries cost the others more: calls of 2047
// inputs, 4 channels, 2100 blocks 135 / 154 at L = 7, 138 / 145 at L = 16.
bool pass_b_direct(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int32_t window, int32_t chunk, int vec) {
  if (window < 2 || (vec != 4 && n_inputs > 64) || n_blocks < 1 || pass_b_scan_free_chunk(n_inputs, n_channels, n_blocks, window)) return false;
  const int W = combine_waves(n_inputs, 4);
  if (W > 1 && n_inputs % 4 == 0) {
    const int64_t waves = n_blocks * n_channels * W;
    const bool runs = runs_suit(n_inputs, window, vec, 1, n_blocks, waves);
    if (n_inputs <= 2048 && (W >= 4 || runs) && waves >= (W >= 4 && runs ? 1 << 15 : 1 << 16)) return false;
    if (n_blocks <= 1152 && window > 16 && waves >= 7 << 12) return false;
  }
  const int64_t rows = window - 1 < n_blocks ? window - 1 : n_blocks;
  const int64_t passes = (n_inputs + 2047) / 2048;
  // (Past 2048 inputs the line is that of two blocks a wavefront, four being no faster:
  // calls of 3000 inputs, 3 channels, 700 blocks, L = 100: 86.0 / 77.9 us.)
  const int64_t wgs = window_workgroups(n_inputs, n_channels, n_blocks, passes > 1 && chunk > 2 ? 2 : chunk);
  return wgs * rows * passes < ((int64_t)1 << (W == 1 ? 18 : 17));
}

size_t pass_b_direct_part_bytes(int32_t n_inputs, int32_t n_channels, int64_t n_blocks) {
  const int W = combine_waves(n_inputs, 4);
  return W > 1 ? (size_t)5 * sizeof(double) * W * n_channels * (size_t)n_blocks : 0;
}

size_t pass_b_direct_done_bytes(int32_t n_inputs, int32_t n_channels, int64_t n_blocks) {
  // Segments of at least 8 blocks.
  return combine_waves(n_inputs, 4) > 1 ? sizeof(uint32_t) * n_channels * (size_t)((n_blocks + 7) / 8) : 0;
}

int32_t pass_b_direct_counts(const PassBArgs& a) {
  const int X = WINDOW_WAVES * a.chunk;
  return a.direct && combine_waves(a.n_inputs, 4) > 1 ? a.n_channels * ((a.n_blocks + X - 1) / X) : 0;
}

// Blocks per wavefront of the window kernel: the fewest that leave at most a
// workgroup per CU (6.4 us at 1 against 7.1 at 2 with 96 workgroups; 9.4 at 2
// against 9.9 at 1 with 256); where 2 still leaves more, 4 if the windows are long
// (13.3 against 14.2 us at L = 256; 14.2 against 12.4 at L = 64).
static int window_chunk(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int32_t window) {
  if (window_workgroups(n_inputs, n_channels, n_blocks, 1) <= 256) return 1;
  if (window_workgroups(n_inputs, n_channels, n_blocks, 2) <= 256 || window <= 128 || n_blocks <= 128) return 2;
  return 4;
}

int pass_b_chunk(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int vec) {
  // Four blocks per combine workgroup, fewer while there are too few
  // wavefronts to fill the device (at least ~4 per SIMD).
  const int64_t waves_per_chunk = combine_waves(n_inputs, vec);
  int R = 4;
  while (R > 1 && ((n_blocks + R - 1) / R) * n_channels * waves_per_chunk < 4096) R /= 2;
  return R;
}


int pass_b_plan_chunk(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int32_t window) {
  const int free_chunk = pass_b_scan_free_chunk(n_inputs, n_channels, n_blocks, window);
  if (free_chunk) return free_chunk;
  const int R = window_chunk(n_inputs, n_channels, n_blocks, window);
  if (pass_b_direct(n_inputs, n_channels, n_blocks, window, R, pass_b_vec(n_inputs))) return R;
  // Runs of 16 blocks cost least at one block a step: fewer registers, and pass A then
  // writes no chunk sums for the scan (whole calls, R = 1 against 4, us: 363.9 / 366.4
  // CHIME M = 256, 206.4 / 211.1 M = 128, 134.8 / 138.4 1024 inputs, 8 channels, M = 64,
  // and windows of 16 k blocks).
  if (runs_suit(n_inputs, window, pass_b_vec(n_inputs), 1, n_blocks, n_blocks * n_channels * combine_waves(n_inputs, 4), true))
    return 1;
  return pass_b_chunk(n_inputs, n_channels, n_blocks, pass_b_vec(n_inputs));
}

size_t pass_b_prefix_bytes(int32_t n_inputs, int32_t n_channels, int64_t n_blocks, int32_t chunk) {
  return (size_t)n_channels * (size_t)((n_blocks + chunk - 1) / chunk + 1) * (size_t)n_inputs * sizeof(uint32_t);
}

__global__ __launch_bounds__(256) void flags_kernel(FlagArgs a) {
#pragma clang fp contract(off)
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= a.n) return;
  const double V = (double)a.v[j];
  const int64_t K = (int64_t)a.n_eff[j] * a.block_len;
  uint8_t fl;
  if (K < 2 || isnan(V) || (a.thresholds && a.n_eff[j] > a.n_max)) {
    fl = SK_FLAG_INVALID;
  } else {
    const double Kd = (double)K, Md = (double)a.block_len;
    double e0 = 1.0;
    if (a.estimator == SK_EST_HAT && a.window == 1) e0 = ((Kd + 1.0) * (Md - 1.0)) / ((Kd - 1.0) * (Md + 1.0));
    const double E = e0 + a.expect_offset;
    const double s = a.sigma_override > 0.0 ? a.sigma_override : sqrt(4.0 / Kd);
    double lo = E - a.k_sigma * s, hi = E + a.k_sigma * s;
    if (a.thresholds) {
      lo = a.thresholds[2 * a.n_eff[j]];
      hi = a.thresholds[2 * a.n_eff[j] + 1];
    }
    fl = (V < lo ? SK_FLAG_LOW : 0) | (V > hi ? SK_FLAG_HIGH : 0);
  }
  a.flags[j] = fl;
}

int launch_flags(const FlagArgs& a, hipStream_t s) {
  if (a.n <= 0) return SK_OK;
  const int64_t grid = (a.n + 255) / 256;
  flags_kernel<<<dim3((unsigned)grid), dim3(256), 0, s>>>(a);
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

}  // namespace sk
