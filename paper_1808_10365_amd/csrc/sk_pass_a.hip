// Pass A: per-input block sums of power and square power (Eq. singlesums).
//
// The input is one byte per complex sample, [T][F][N] (time-major, inputs
// innermost). Each lane owns VEC consecutive inputs of one channel and walks
// the rows (time samples) of a block with one VEC-byte nontemporal load per
// row, so a wavefront reads 64*VEC contiguous bytes per row. Power comes from
// an LDS table indexed by the byte (Re and Im decoded from the nibbles,
// Sec. 2.2.3 "Calculating Power"). Sums are exact in 32 bits: p <= 128, so
// S2 <= M * 2^14 < 2^31 for M <= 131071.
//
// Variants (sk_profile.h):
//   0 shared 256-entry table of p; two rows' powers packed into the 16-bit
//     halves of a register so v_dot2_u32_u16 adds p0^2 + p1^2 to S2 and
//     p0 + p1 to S1; a workgroup of 256 lanes covers LPR column groups times
//     256 / LPR row phases, reduced in LDS. Any vector width (16, 4, 1).
//   1, 2 packed lane-replicated table (entries p | p^2 << 12, one add per
//     sample for both sums), one row phase of 256..1024 lanes, 8 or 16 rows
//     per load.
//   3 packed table, 256-lane workgroups whose lanes sum whole rows; narrow
//     rows put 256 / L blocks side by side.
//   4 packed table, 512-lane workgroups walking up to 4 consecutive blocks
//     with every block's sums held in registers and stored at the task's end.
//   5 packed table, 512-lane workgroups of row phases over runs of 16-byte units,
//     any N and alignment (library choice only).
//   6 the same from aligned dwords, for rows off 4-byte boundaries (library choice
//     only).
#include <hip/hip_runtime.h>

#include "sk_internal.h"
#include "sk_pass_a_dev.h"
#include "sk_wave_dev.h"

namespace sk {

// Workgroup size: 256 lanes, or LPR lanes (512, 1024) when a workgroup spans
// a whole wide row with one row phase (one contiguous slab per block).
template <int LPR>
constexpr int wg_size() { return LPR > 256 ? LPR : 256; }

// Stores one lane's sums of column group g (VEC inputs) for block b.
template <int VEC>
__device__ __forceinline__ void store_group(const PassATask& t, int b, int g, const uint32_t* s1,
                                            const uint32_t* s2) {
  const int N = t.n_inputs;
  const int B = t.n_blocks;
  const int64_t col = (int64_t)g * VEC;
  const int64_t f = col / N, i = col % N;
  int32_t* d1 = t.s1 + (f * B + b) * N + i;
  int32_t* d2 = t.s2 + (f * B + b) * N + i;
  if constexpr (VEC >= 4) {
#pragma unroll
    for (int k = 0; k < VEC; k += 4) {
      u32x4 a = {s1[k], s1[k + 1], s1[k + 2], s1[k + 3]};
      u32x4 c = {s2[k], s2[k + 1], s2[k + 2], s2[k + 3]};
      // Plain stores: nontemporal ones measured far slower here (the sums
      // then reach HBM as scattered partial writes).
      *reinterpret_cast<u32x4*>(d1 + k) = a;
      *reinterpret_cast<u32x4*>(d2 + k) = c;
    }
  } else {
    d1[0] = (int32_t)s1[0];
    d2[0] = (int32_t)s2[0];
  }
}

// Variant 0: shared table. One task is (block b, chunk ch) of LPR column
// groups; lane lc of row phase ph owns group ch * LPR + lc, so a wavefront's
// loads of one row are 64 * VEC contiguous bytes. The row phases' partial
// sums meet in LDS (VEC words of S1 then VEC of S2 per lane, odd stride).
template <int VEC, int LPR>
__global__ __launch_bounds__(wg_size<LPR>()) void pass_a_shared_kernel(PassATask t) {
  constexpr int WG = wg_size<LPR>();
  constexpr int RP = WG / LPR;          // row phases per workgroup
  constexpr int W = 2 * VEC + 1;        // LDS stride of one lane's partials (odd: no bank conflicts)
  constexpr int U = 8;                  // rows per load batch
  __shared__ uint16_t lut16[256];
  extern __shared__ uint32_t red[];     // [RP * LPR][W] when RP > 1
  const int tid = threadIdx.x;
  for (int k = tid; k < 256; k += WG) lut16[k] = (uint16_t)code_power((uint32_t)k);
  __syncthreads();
  const CountsToClear<WG> counts(t);
  const int lc = tid % LPR;
  const int ph = tid / LPR;
  const int M = t.block_len;
  const int64_t G = t.row_bytes;
  for (int64_t task = blockIdx.x; task < t.n_tasks; task += gridDim.x) {
    const int b = t.block0 + (int)(task / t.chunks);
    const int ch = (int)(task % t.chunks);
    const int g0 = ch * LPR + lc;
    uint32_t s1[VEC], s2[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) s1[k] = s2[k] = 0;
    if (g0 < t.col_groups)
      sum_rows<VEC, RP, U>(t.x + (int64_t)b * M * G + (int64_t)g0 * VEC, G, M, ph, lut16, s1, s2);
    if constexpr (RP == 1) {
      if (g0 < t.col_groups) store_group<VEC>(t, b, g0, s1, s2);
    } else {
      const int N = t.n_inputs;
      const int B = t.n_blocks;
      uint32_t* mine = red + (ph * LPR + lc) * W;
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        mine[k] = s1[k];
        mine[VEC + k] = s2[k];
      }
      __syncthreads();
      for (int o = tid; o < LPR * 2 * VEC; o += WG) {
        const int l = o / (2 * VEC), k = o % (2 * VEC);
        uint32_t s = 0;
#pragma unroll 8
        for (int q = 0; q < RP; ++q) s += red[(q * LPR + l) * W + k];
        const int gg = ch * LPR + l;
        if (gg < t.col_groups) {
          const int64_t col = (int64_t)gg * VEC + (k % VEC);
          const int64_t f = col / N, i = col % N;
          int32_t* dst = k < VEC ? t.s1 : t.s2;
          dst[(f * B + b) * N + i] = (int32_t)s;
        }
      }
      __syncthreads();
    }
  }
  counts.clear(tid);
}

template <int VEC, int LPR>
static int launch_shared_one(const PassATask& t, int grid, hipStream_t s, PassEvents ev) {
  constexpr int WG = wg_size<LPR>();
  constexpr int RP = WG / LPR;
  const size_t lds = RP > 1 ? sizeof(uint32_t) * WG * (2 * VEC + 1) : 0;
  launch_kernel(pass_a_shared_kernel<VEC, LPR>, dim3(grid), dim3(WG), (uint32_t)lds, s, ev.start, ev.stop, t);
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

template <int VEC>
static int launch_shared(const PassATask& t, int lpr, int grid, hipStream_t s, PassEvents ev) {
  switch (lpr) {
    case 1: return launch_shared_one<VEC, 1>(t, grid, s, ev);
    case 2: return launch_shared_one<VEC, 2>(t, grid, s, ev);
    case 4: return launch_shared_one<VEC, 4>(t, grid, s, ev);
    case 8: return launch_shared_one<VEC, 8>(t, grid, s, ev);
    case 16: return launch_shared_one<VEC, 16>(t, grid, s, ev);
    case 32: return launch_shared_one<VEC, 32>(t, grid, s, ev);
    case 64: return launch_shared_one<VEC, 64>(t, grid, s, ev);
    case 128: return launch_shared_one<VEC, 128>(t, grid, s, ev);
    case 256: return launch_shared_one<VEC, 256>(t, grid, s, ev);
    case 512: return launch_shared_one<VEC, 512>(t, grid, s, ev);
    case 1024: return launch_shared_one<VEC, 1024>(t, grid, s, ev);
  }
  set_error("pass A: unsupported lanes-per-row %d", lpr);
  return SK_ERR_INVALID_ARG;
}

// Variants 1 and 2: packed lane table, one row phase of LPR lanes (256, 512
// or 1024). A task walks blocks_per_task consecutive blocks (contiguous
// rows) of one column chunk, storing each block's sums as it ends.
template <int LPR, int U>
__global__ __launch_bounds__(LPR) void pass_a_packed_kernel(PassATask t) {
  constexpr int VEC = 16;
  __shared__ __attribute__((aligned(16))) uint32_t lut32[LANE_LUT_DWORDS];
  const int tid = threadIdx.x;
  fill_lane_packed_lut<LPR>(lut32, tid);
  __syncthreads();
  const CountsToClear<LPR> counts(t);
  const LanePackedLut lut{reinterpret_cast<const uint8_t*>(lut32), (uint32_t)(tid & 63) * 4};
  const int M = t.block_len;
  const int64_t G = t.row_bytes;
  const int Q = t.blocks_per_task;
  for (int64_t task = blockIdx.x; task < t.n_tasks; task += gridDim.x) {
    const int b_first = t.block0 + (int)(task / t.chunks) * Q;
    const int g0 = (int)(task % t.chunks) * LPR + tid;
    if (g0 >= t.col_groups) continue;
    for (int b = b_first; b < b_first + Q && b < t.block_end; ++b) {
      uint32_t s1[VEC], s2[VEC];
#pragma unroll
      for (int k = 0; k < VEC; ++k) s1[k] = s2[k] = 0;
      sum_rows_packed<VEC, 1, U>(t.x + (int64_t)b * M * G + (int64_t)g0 * VEC, G, M, 0, lut, s1, s2);
      store_group<VEC>(t, b, g0, s1, s2);
    }
  }
  counts.clear(tid);
}

template <int U>
static int launch_packed(const PassATask& t, int lpr, int grid, hipStream_t s, PassEvents ev) {
  switch (lpr) {
    case 256: launch_kernel(pass_a_packed_kernel<256, U>, dim3(grid), dim3(256), 0, s, ev.start, ev.stop, t); break;
    case 512: launch_kernel(pass_a_packed_kernel<512, U>, dim3(grid), dim3(512), 0, s, ev.start, ev.stop, t); break;
    case 1024: launch_kernel(pass_a_packed_kernel<1024, U>, dim3(grid), dim3(1024), 0, s, ev.start, ev.stop, t); break;
    default:
      set_error("pass A: packed lane-table variant needs 256..1024 lanes per row, got %d", lpr);
      return SK_ERR_INVALID_ARG;
  }
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

// Variant 3: packed lane table, 256-lane tasks with blocks side by side for
// narrow rows (t.blocks_per_task blocks per task) or 256-group chunks of one
// block for wide rows; no row phases, so no reduction across lanes.
template <int U>
__global__ __launch_bounds__(256) void pass_a_side_by_side_kernel(PassATask t, int lpb) {
  __shared__ __attribute__((aligned(16))) uint32_t lut32[LANE_LUT_DWORDS];
  const int tid = threadIdx.x;
  fill_lane_packed_lut<256>(lut32, tid);
  __syncthreads();
  const CountsToClear<256> counts(t);
  const LanePackedLut lut{reinterpret_cast<const uint8_t*>(lut32), (uint32_t)(tid & 63) * 4};
  for (int64_t task = blockIdx.x; task < t.n_tasks; task += gridDim.x)
    pass_a_task_side_by_side<U>(t, lpb, task, lut, tid);
  counts.clear(tid);
}

int pass_a_side_by_side_lanes(int64_t col_groups) {
  int lpb = 1;
  while (lpb < 256 && lpb < col_groups) lpb *= 2;
  return lpb;
}

// Variant 4: packed table, 512-lane workgroups over chunks of 512 column
// groups; a task walks Q consecutive blocks holding every block's sums in
// registers and stores them only after its last block. With about one task
// per CU the call becomes a read phase followed by a write phase: mixing
// the sums' writes into the read stream costs far more than their bytes
// (CHIME M = 256: 335 against 382 us with a store after each block). The
// two wavefronts of each SIMD keep level through SimdBalance.
//
// With t.timeline set (one task per workgroup), lane 0 of every wavefront
// records the real-time clock (100 MHz) at its start, after its reads (the
// stamp depends on the sums, so it follows the last load) and after its
// stores have completed, then its XCD and HW_ID registers, at
// timeline[6 (8 blockIdx.x + wavefront) ...]. BAL = false leaves the
// wavefronts of a SIMD to the arbiter (for timelines that compare).
template <int Q, int U, bool BAL = true>
__global__ __launch_bounds__(512) void pass_a_deferred_kernel(PassATask t) {
  constexpr int VEC = 16;
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
  __shared__ __attribute__((aligned(16))) uint32_t lut32[LANE_LUT_DWORDS];
  __shared__ uint32_t simd_of[8], progress[8];
  const int tid = threadIdx.x;
  fill_lane_packed_lut<512>(lut32, tid);
  simd_balance_post(simd_of, progress, tid);
  __syncthreads();
  const CountsToClear<512> counts(t);
  SimdBalance bal = simd_balance_pair(simd_of, progress, 8);
  NoBalance arbiter;
  const LanePackedLut lut{reinterpret_cast<const uint8_t*>(lut32), (uint32_t)(tid & 63) * 4};
  const int M = t.block_len;
  const int64_t G = t.row_bytes;
  uint64_t t_reads = 0;
  for (int64_t task = blockIdx.x; task < t.n_tasks; task += gridDim.x) {
    const int b0 = t.block0 + (int)(task / t.chunks) * Q;
    const int g = (int)(task % t.chunks) * 512 + tid;
    if (g >= t.col_groups) continue;
    uint32_t a1[Q][VEC], a2[Q][VEC];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
#pragma unroll
      for (int k = 0; k < VEC; ++k) a1[q][k] = a2[q][k] = 0;
      if (b0 + q < t.block_end) {
        const uint8_t* base = t.x + (int64_t)(b0 + q) * M * G + (int64_t)g * VEC;
        if constexpr (BAL) sum_rows_packed<VEC, 1, U>(base, G, M, 0, lut, a1[q], a2[q], bal);
        else sum_rows_packed<VEC, 1, U>(base, G, M, 0, lut, a1[q], a2[q], arbiter);
      }
    }
    if (t.timeline) {
      uint32_t dep = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) dep |= a1[q][0] >> 31;
      t_reads = __builtin_amdgcn_s_memrealtime() + __builtin_amdgcn_readfirstlane(dep);
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (b0 + q < t.block_end) store_group<VEC>(t, b0 + q, g, a1[q], a2[q]);
    if (t.cs) {
      // S1 over the task's blocks: the chunk sums pass B's prefix scan reads
      // instead of the rows (blocks past the end hold zero sums).
      uint32_t c[VEC];
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        c[k] = a1[0][k];
#pragma unroll
        for (int q = 1; q < Q; ++q) c[k] += a1[q][k];
      }
      const int N = t.n_inputs;
      const int64_t col = (int64_t)g * VEC;
      const int64_t f = col / N, i = col % N;
      const int64_t nk = (t.n_blocks + Q - 1) / Q;
      int32_t* d = t.cs + (f * nk + (b0 - t.block0) / Q) * N + i;
#pragma unroll
      for (int k = 0; k < VEC; k += 4) *reinterpret_cast<u32x4*>(d + k) = u32x4{c[k], c[k + 1], c[k + 2], c[k + 3]};
    }
  }
  counts.clear(tid);
  if (t.timeline) {
    __builtin_amdgcn_s_waitcnt(0);
    const uint64_t t_end = __builtin_amdgcn_s_memrealtime();
    if ((tid & 63) == 0) {
      uint64_t* o = t.timeline + ((int64_t)blockIdx.x * 8 + (tid >> 6)) * 6;
      o[0] = t_start;
      o[1] = t_reads;
      o[2] = t_end;
      o[3] = (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11));   // XCC_ID bits 3:0
      o[4] = (uint32_t)__builtin_amdgcn_s_getreg(4 | (31 << 11));   // HW_ID
      o[5] = simd_id();
    }
  }
}

// Variant 5 (library choice only): packed lane table with row phases, any N and
// any alignment. A unit is 16 consecutive bytes of a row over one block (they
// may straddle two channels); when 16 does not divide the row, its last unit is
// moved back to end with the row, and the columns it shares with its neighbour
// are summed by both. A workgroup takes LPR consecutive units (over block ends)
// times 512 / LPR row phases, so no lane idles at a row's end and a call of few
// blocks still has many loads in flight. The first rows are in flight while the
// table is filled, and each batch of rows is loaded before the batch ahead of it
// is summed.
//
// The phases meet in LDS: the row groups of a wavefront first (two swaps leave
// each lane 8 of the 32 sums at LPR = 16, as in the combine), then one LDS add
// per value left.
//
// Bound by HBM for calls of about 50 MB to 0.5 GB, at 80 to 93 % of the read
// ceiling: 1000 inputs, 3 channels, 98 MB 31.7 -> 18.8 us (5.2 TB/s; 4-byte lanes
// before), 2048 inputs, 403 MB 68 -> 61 us (6.6 TB/s), 1024 inputs, 268 MB 51 ->
// 43 us (6.2 TB/s; one wavefront per SIMD before), 256 inputs, 50 MB 13.8 -> 11.5
// us (the shared table's bank conflicts before).
template <int LPR>
__global__ __launch_bounds__(512, 4) void pass_a_phased_kernel(PassATask t) {
  constexpr int S = phased_stride(LPR);
  // The sums where the phases meet, in the table's place where they would cost a
  // second workgroup per CU.
  constexpr bool OVER = LPR > 64, RED = !OVER && LPR < 512;
  __shared__ __attribute__((aligned(16))) uint32_t lut32[LANE_LUT_DWORDS];
  __shared__ uint32_t red_own[RED ? 32 * S : 1];
  const int tid = threadIdx.x;
  const CountsToClear<512> counts(t);
  const LanePackedLut lut{reinterpret_cast<const uint8_t*>(lut32), (uint32_t)(tid & 63) * 4};
  pass_a_task_phased<LPR, OVER, false>(t, pass_a_task_of(t) * LPR, lut, OVER ? lut32 : red_own, tid, [&] {
    fill_lane_packed_lut<512>(lut32, tid);
    if constexpr (RED)
      for (int o = tid; o < 32 * S; o += 512) red_own[o] = 0u;
    lds_barrier();
  });
  counts.clear(tid);
}

static int launch_phased(const PassATask& t, int lpr, int grid, hipStream_t s, PassEvents ev) {
  const dim3 g(grid), w(512);
  switch (lpr) {
    case 16: launch_kernel(pass_a_phased_kernel<16>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 32: launch_kernel(pass_a_phased_kernel<32>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 64: launch_kernel(pass_a_phased_kernel<64>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 128: launch_kernel(pass_a_phased_kernel<128>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 256: launch_kernel(pass_a_phased_kernel<256>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 512: launch_kernel(pass_a_phased_kernel<512>, g, w, 0, s, ev.start, ev.stop, t); break;
    default:
      set_error("pass A: phased variant needs 16..512 lanes per row, got %d", lpr);
      return SK_ERR_INVALID_ARG;
  }
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

// Variant 6 (library choice only): row phases for rows that do not keep to 4-byte
// boundaries. The phases are a multiple of four, so all rows of a lane start at the
// same place within a dword, and the lane reads its 16 bytes from the aligned dword
// at or before its unit: whole 16-byte loads of dwords, where the hardware splits
// loads off a dword boundary, and byte loads cost a lane per column. The windows of
// different phases lie up to 3 columns apart, so the phases meet in LDS column by
// column, and a workgroup reads one unit more than it stores for the columns that
// shifted windows of the next unit hold. Only aligned dwords that hold a byte of the
// frame are read. 3003-byte rows, M = 256, 98 MB: 25 -> 20 us (5.0 TB/s, as rows of
// 3000 bytes); M = 128, 0.4 GB: 95 -> 77; 65 MB of 2545-byte rows 20 -> 13.4. Bound by
// the lines that the ends of a workgroup's rows share with others', and at short
// blocks by the rows a last batch masks.
template <int LPR>
__global__ __launch_bounds__(512, 4) void pass_a_shifted_kernel(PassATask t) {
  constexpr int S = shifted_stride(LPR);
  __shared__ __attribute__((aligned(16))) uint32_t lut32[LANE_LUT_DWORDS];
  __shared__ uint32_t red[32 * S];
  const int tid = threadIdx.x;
  const CountsToClear<512> counts(t);
  const LanePackedLut lut{reinterpret_cast<const uint8_t*>(lut32), (uint32_t)(tid & 63) * 4};
  pass_a_task_shifted<LPR>(t, pass_a_task_of(t) * (LPR - 1), lut, red, tid, [&] {
    fill_lane_packed_lut<512>(lut32, tid);
    for (int o = tid; o < 32 * S; o += 512) red[o] = 0u;
    lds_barrier();
  });
  counts.clear(tid);
}

static int launch_shifted(const PassATask& t, int lpr, int grid, hipStream_t s, PassEvents ev) {
  const dim3 g(grid), w(512);
  switch (lpr) {
    case 16: launch_kernel(pass_a_shifted_kernel<16>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 32: launch_kernel(pass_a_shifted_kernel<32>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 64: launch_kernel(pass_a_shifted_kernel<64>, g, w, 0, s, ev.start, ev.stop, t); break;
    case 128: launch_kernel(pass_a_shifted_kernel<128>, g, w, 0, s, ev.start, ev.stop, t); break;
    default:
      set_error("pass A: shifted variant needs 16..128 lanes per row, got %d", lpr);
      return SK_ERR_INVALID_ARG;
  }
  SK_HIP_TRY(hipGetLastError());
  return SK_OK;
}

// Blocks per task for variant 4: about one task per CU, at most 4 (the
// sums of 4 blocks take 128 registers per lane).
int pass_a_deferred_blocks(int64_t n_blocks, int64_t col_groups, int n_cu) {
  const int64_t chunks = (col_groups + 511) / 512;
  int64_t q = (n_blocks * chunks + n_cu - 1) / (n_cu > 0 ? n_cu : 1);
  return (int)(q < 1 ? 1 : (q > 4 ? 4 : q));
}

bool pass_a_packed(int vec, int variant) { return vec == 16 && (variant == 1 || variant == 2); }

bool pass_a_side_by_side(int vec, int variant) { return vec == 16 && variant == 3; }

bool pass_a_deferred(int vec, int variant) { return vec == 16 && variant == 4; }

void pass_a_lane_range(int vec, int variant, int* lo, int* hi) {
  *lo = 1;
  *hi = 1024;
  if (vec != 16 || variant == 0) return;
  if (variant == 3) { *lo = 1; *hi = 256; }
  else if (variant == 4) { *lo = 512; *hi = 512; }
  else { *lo = 256; }
}

template <int VEC>
static int launch_vec(const PassATask& t, int lpr, int variant, int grid, hipStream_t s, PassEvents ev) {
  if constexpr (VEC == 16) {
    const dim3 g(grid), w512(512);
    switch (variant) {
      case 1: return launch_packed<8>(t, lpr, grid, s, ev);
      case 5: return launch_phased(t, lpr, grid, s, ev);
      case 6: return launch_shifted(t, lpr, grid, s, ev);
      case 2: return launch_packed<16>(t, lpr, grid, s, ev);
      case 3:
        launch_kernel(pass_a_side_by_side_kernel<16>, g, dim3(256), 0, s, ev.start, ev.stop, t, lpr);
        SK_HIP_TRY(hipGetLastError());
        return SK_OK;
      case 4:
        switch (t.blocks_per_task) {
          case 1: launch_kernel(pass_a_deferred_kernel<1, 16>, g, w512, 0, s, ev.start, ev.stop, t); break;
          case 2: launch_kernel(pass_a_deferred_kernel<2, 16>, g, w512, 0, s, ev.start, ev.stop, t); break;
          case 3: launch_kernel(pass_a_deferred_kernel<3, 16>, g, w512, 0, s, ev.start, ev.stop, t); break;
          case 4:
            if (t.simd_balance) launch_kernel(pass_a_deferred_kernel<4, 16>, g, w512, 0, s, ev.start, ev.stop, t);
            else launch_kernel(pass_a_deferred_kernel<4, 16, false>, g, w512, 0, s, ev.start, ev.stop, t);
            break;
          default:
            set_error("pass A: deferred-store variant needs 1..4 blocks per task, got %d", t.blocks_per_task);
            return SK_ERR_INVALID_ARG;
        }
        SK_HIP_TRY(hipGetLastError());
        return SK_OK;
      default: break;
    }
  }
  return launch_shared<VEC>(t, lpr, grid, s, ev);
}

// Two workgroups fit a CU: with somewhat more than one each, some CUs have twice the
// others' work (2044 inputs, 2 channels, 314 MB: 68 us with 300, 58 with 600).
static bool uneven_workgroups(int64_t n, int n_cu) { return n > n_cu && 32 * n < 55 * (int64_t)n_cu; }

// Rows of dwords off 16-byte boundaries in which variant 0, whose lanes take a dword each,
// is faster than variant 5 though that keeps more loads in flight: calls of many units,
// where its 16-byte loads are split or `rows`, a block's rows in whole batches, are many
// more than M; and narrow rows, whose blocks are apart. Measured, variant 0 / 5 (us):
//   32 bytes 69 / 74 (M = 160, 200 MB), 68 / 87 (M = 1024, 390 MB), but 73 / 59 (M = 128);
//   48 bytes 83 / 100 (M = 2000, 400 MB), but 59 / 55 with 36 (M = 1757, 241 MB); 64 bytes 10.1 / 13.4 (M = 140, 30 MB);
//   80 bytes 53 / 61 (M = 140, 114 MB); 112 bytes 11.1 / 12.2 (M = 64, 30 MB);
//   240 bytes 20.4 / 25.4 (M = 64, 80 MB; 12.4 / 11.8 with 30 MB), 44 / 49 (M = 100, 200 MB);
//   256 bytes 37 / 48 (M = 256, 200 MB), 75 / 93 (M = 512, 400 MB; 61 / 44 with 200 MB);
//   512 bytes 20.8 / 25.3 (M = 50, 80 MB; 56 is the better in variant 5).
// (4268 calls of 27 row lengths, 3 to 350 MB: of the 490 that this moves, 23 lose 5 % or
// more, all are 9 % faster on average.)
static bool dword_rows_shared(int64_t row_bytes, int64_t units, int M, int rows) {
  const int64_t cg = (row_bytes + 15) / 16;
  auto in = [&](int above, int to) { return M > above && M <= to; };
  if (cg == 2) return in(64, 100) || (M > 130 && !(in(180, 400) && units >= 22000));
  if (cg == 3)
    return (in(64, 100) && units < 12000) || (in(200, 400) && units < 5000) || (row_bytes > 40 && M >= 1400 && units >= 8000);
  if (cg == 4)
    return (in(64, 100) && units < 12000) || in(130, 200) || (in(200, 400) && units >= 5000) || (M >= 1400 && units >= 8000);
  if (cg >= 5 && cg < 10 && M > 64 && units >= 12000 && 2 * rows > 3 * M) return true;
  if (cg == 5) return in(70, 85) && units >= 12000;
  if (cg >= 6 && cg < 9)
    return (in(60, 85) && units >= 12000) || (in(85, 130) && units >= 24000) || (in(30, 60) && units >= 16000 && units < (M > 45 ? 100000 : 1 << 15)) ||
           (in(130, 180) && units >= 12000) || (in(180, 260) && units >= 24000);
  if (cg >= 9 && cg < 12) return (in(30, 60) && units >= 24000 && units < 140000) || (in(60, 105) && units >= 33000);
  if (cg >= 12 && cg < 18)
    return (in(30, 260) && units >= (M <= 45 && cg < 16 ? 24000 : 33000)) ||
           (cg >= 16 && in(260, 800) && units >= 33000 && units < (M < 400 ? 130000 : 60000));
  return cg >= 18 && cg < 64 && in(30, 60) && units >= 65000 && units < 105000 && 4 * rows > 5 * M;
}

// Units a workgroup of variant 5 takes for a call it suits, else 0. Measured,
// pass A alone (us, variant 5 against the best other):
//   rows not of 16-byte groups, on 4-byte boundaries: 20.2 / 31.7 (3000 bytes,
//     M = 256, 98 MB), 92 / 128 (4004 bytes, 525 MB), 39 / 38.5 at M = 16, 57 / 40
//     at M = 2: from 16 rows a block;
//   off 4-byte boundaries, where the hardware splits the loads: 24 / 29 (3003
//     bytes, M = 256), 51 / 70 (2047 bytes, M = 256), 21.6 / 18.8 (2545 bytes,
//     M = 100), 12.7 / 9.5 (17 bytes): from 192 rows and 256 bytes;
//   16-byte groups: 61 / 68 (2048 inputs, 403 MB), 43 / 51 (1024 inputs, 268 MB),
//     11.5 / 13.8 (256 inputs, 50 MB), 21 / 65 (16 inputs, 67 MB), but 175 / 174 at
//     1 GiB, 360 / 334 at 2 GiB, 98 / 95 at 0.5 GiB of M = 128 and 105 / 102 for wide
//     rows of M = 64: the variants whose lanes hold whole rows there;
//   little work: 5.5 / 5.3 below 1024 units, 6.7 / 4.2 in short blocks of 2 MB, and in
//     narrow rows 6.4 / 5.6 (16 bytes, M = 256, 8 MB);
//   long blocks in narrow rows, 16 units a workgroup, where that gives few workgroups or a few
//     past one per CU: 20.8 / 12.7 (16 bytes, M = 1700, 1102 units), 26.0 / 19.5 (M = 900,
//     4166), 18.2 / 15.6 (32 bytes, 4166); 15.2 / 17.0 between (16 bytes, M = 1024, 3662);
//   narrow rows off 16-byte boundaries: 106 / 68 (16 bytes, M = 640, 300 MB), 43 / 39 (M =
//     160, 70 MB), 298 / 238 (M = 80, 300 MB); 56.8 / 52.4 (48 bytes, M = 160, 200 MB);
//     34.9 / 32.5 (64 bytes, M = 128, 130 MB), 61.5 / 58.4 (M = 256, 300 MB); 71.5 / 63.7
//     (104 bytes, M = 200, 300 MB); 129 / 118 (144 bytes, M = 160, 500 MB);
//   short blocks: 17.0 / 14.0 (200 bytes, M = 24, 30 MB), 135 / 116 (600 bytes, M = 20, 500
//     MB), 20.5 / 17.0 (4000 bytes, M = 20, 45 MB; 11.0 / 13.6 with 20 MB), 135 / 124 (352
//     bytes, M = 50, 500 MB), 12.3 / 10.6 (4000 bytes, M = 34, 20 MB); where the last
//     batch is mostly masked 23.4 / 21.0 (104 bytes, M = 90), 30.8 / 24.8 (160 inputs, M = 80,
//     100 MB); and where 55 / 47 side by side (64 inputs, M = 40, 130 MB), but 26.5 / 41.4
//     (400 inputs, 4 channels, M = 60).
int pass_a_phased_lanes(const uint8_t* x, int64_t row_bytes, int32_t n_inputs, int64_t n_blocks, int block_len, int n_cu) {
  const int64_t cg = (row_bytes + 15) / 16, units = cg * n_blocks;
  const int M = block_len;
  // 24-bit row bytes and 32-bit offsets over the blocks a workgroup spans.
  if (row_bytes < 16 || row_bytes >= (1 << 24) || units < 1024 || units >= ((int64_t)1 << 30) ||
      (512 / cg + 2) * M * row_bytes >= ((int64_t)1 << 31))
    return 0;
  const bool whole = pick_vec(x, n_inputs) == 16;
  // A few workgroups of 16 units past one per CU.
  const bool past_cu = units > 16 * (int64_t)n_cu && 16 * units < 325 * (int64_t)n_cu;
  if (whole) {
    if (M < 32 || units * M * 16 > ((int64_t)1 << (M < 192 ? 28 : 29)) || (cg >= 512 && M < 128) ||
        (cg >= 2 && cg < 10 && M < 50 && units >= 1 << 16) ||
        (cg == 1 && ((M >= 900 && units < 1900) || (M >= 1600 && units > 4096 && units < 7040) || (M >= 2500 && units < 3000))) ||
        (cg == 3 && ((M >= 1024 && units < 1600) || (M >= 2500 && past_cu))))
      return 0;
  } else if (row_bytes % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 4 == 0) {
    if (M < 16 || (cg <= 4 && (units < 2048 || (M >= 640 && past_cu))) || (cg == 1 && M >= 640 && (units < 2240 || (units > 4096 && units < 5800))) ||
        (cg == 1 && M > 128 && reinterpret_cast<uintptr_t>(x) % 16) ||
        (cg == 3 && M > 128 && M < 192) || (cg == 4 && M >= 128 && M < 512 && units >= 1 << 14) ||
        ((cg == 6 || cg == 7) && M >= 128 && M < 256 && units >= 1 << 15) ||
        (cg >= 8 && cg < 12 && M >= 128 && M < 192 && units >= 1 << 17) ||
        (cg >= 12 && cg < 64 && M < 32 && units >= 1 << 16) ||
        (cg >= 16 && M < 40 && ((units >= 96000 && units < 160000) || (M >= 32 && units >= 30000 && units < 60000))) ||
        (cg >= 16 && cg < 48 && M >= 44 && M < 64 && units >= 1 << 17))
      return 0;
  } else if (M < 192 || cg < 16) {
    return 0;
  }
  if (M > 16 && M < 64 && units * M * 16 < 3 << 20 && !(whole && cg <= 3)) return 0;
  // About one workgroup per CU (256 in these figures) with the fewest phases to join (in1000: 20.2 us
  // with 188 workgroups of 128 units, 21.4 with 752 of 32, 29 with 94 of 256); rows of
  // under 16 groups keep a wavefront's lanes on neighbouring rows, and short calls
  // take 16 units (within a microsecond of the best there). Where a block is but one or two
  // batches of rows, fewer phases waste fewer: 32 units at 128 to 191 rows (104 bytes,
  // 130 MB: 31.4 us, 38.3 with 16; 352 bytes, 300 MB: 65, 78 with 256) and at 33 to 63
  // rows (32 bytes, 130 MB: 63.5, 83 with 64) unless there are many wide units (200
  // bytes, 300 MB: 88 with 512, 119 with 32).
  int lanes = 16;
  if (cg >= 16 && units >= (1 << 14)) {
    while (lanes < (M < 128 ? (M >= 64 && cg < 32 ? 128 : 256) : M < 192 && cg < 32 ? 64 : 512) && 5 * (int64_t)n_cu / 8 * 2 * lanes <= units) lanes *= 2;
    if (lanes > 32 && uneven_workgroups(units / lanes, n_cu)) lanes /= 2;
  } else if (cg >= 6 && M > 32 && M < 64 && units >= 1 << 15) {
    lanes = units >= 3 << 16 ? 512 : 256;
  } else if (cg >= 6 && M >= 128 && M < 192 && units >= 1 << 13) {
    lanes = 32;
  }
  // At least 4 rows a lane; no further than 32 units in the narrow rows above.
  while (lanes < 256 && lanes * M < 2048 && !(M > 32 && lanes >= 32 && cg < 6 && units >= 1 << 12)) lanes *= 2;
  // Rows in whole batches against the block's own.
  const int batch = 2048 / lanes, rows = (M + batch - 1) / batch * batch;
  const bool much = M >= 64 && M < 100 && 10 * rows > 13 * M;
  if (whole) {
    if (much && cg >= 6 && cg < 16 && units >= 1 << 16) return 0;
  } else if (cg == 1) {
    if (much && reinterpret_cast<uintptr_t>(x) % 16) return 0;
  } else if (cg >= 6 && cg < 16 && units >= 1 << 15 && (much || (M < 64 && 10 * rows > 11 * M))) {
    return 0;
  }
  if (!whole && row_bytes % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 4 == 0 && dword_rows_shared(row_bytes, units, M, rows)) return 0;
  return lanes;
}

// Units a workgroup of variant 6 takes for a call it suits, else 0. Measured, pass A
// alone (us, variant 6 against the best other):
//   20 / 25 (3003 bytes, M = 256, 98 MB), 13 / 19 (2545 bytes, M = 256, 65 MB), 14 / 27
//     (202 bytes, M = 1000, 26 MB), 8 / 13 (297 bytes, M = 150), 6.6 / 12.5 (129
//     bytes, M = 256), 77 / 95 (3003 bytes, M = 128, 0.4 GB), 5.1 / 6.7 (602 bytes, M =
//     128, 4.6 MB); 5.6 / 4.2 below 4 MB (297 bytes, M = 128); rows of under 8 units
//     66 / 37 (47 bytes, M = 1100);
//   short blocks only in wide rows and where there are many: 217 / 255 (2545 bytes, M =
//     100, 1 GB), 57 / 64 (4095 bytes, M = 64, 262 MB), but 19.1 / 19.1 with 65 MB of
//     the first, 40.6 / 40 (131 bytes, M = 64) and 10 / 8.4 (189 bytes, M = 64);
//   long blocks of wide rows stay with variant 5 where its workgroups of 256 units are just short of one
//     per CU: 51 / 53 (2047 bytes, M = 256, 262 MB), 68 / 64 (M = 320);
//   many units of blocks of 256 or 320 rows in narrow rows stay with variant 5: 109 / 97
//     (450 bytes, M = 256, 500 MB), 80 / 72 (350 bytes, M = 320, 330 MB), but 83 / 124 with
//     M = 192 (1000 bytes, 420 MB), 85 / 95 (2047 bytes, M = 256, 420 MB), 102 / 108 (350
//     bytes, M = 512, 500 MB); and the narrowest rows with variant 0: 43.3 / 37.1 (117
//     bytes, M = 128, 130 MB), 41.4 / 31.9 (123 bytes, M = 392), 37.5 / 26.3 (128 bytes, M =
//     256, 131 MB).
int pass_a_shifted_lanes(const uint8_t* x, int64_t row_bytes, int64_t n_blocks, int block_len, int n_cu) {
  const int64_t cg = (row_bytes + 18) / 16, units = cg * n_blocks;
  if (row_bytes % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 4 == 0) return 0;
  if (cg < (block_len < 128 ? 64 : 8) || block_len < 64 || units < (block_len < 128 ? 1 << 17 : 1024) ||
      units * block_len < 1 << 18 || (cg <= 9 && units > 15000) ||
      (block_len >= 192 && units > 60000 && ((cg >= 64 && units <= 256 * (int64_t)n_cu) || (block_len > 240 && block_len < 400 && cg >= 16 && cg < 32))) ||
      row_bytes >= (1 << 24) || units >= ((int64_t)1 << 30) || (512 / cg + 2) * block_len * row_bytes >= ((int64_t)1 << 31))
    return 0;
  int lanes = 16;
  while (lanes < 128 && 128 * (units / (2 * lanes - 1)) >= 75 * (int64_t)n_cu) lanes *= 2;
  return lanes > 16 && uneven_workgroups(units / (lanes - 1), n_cu) ? lanes / 2 : lanes;
}

int pick_vec(const uint8_t* x, int32_t n_inputs) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(x);
  if (n_inputs % 16 == 0 && a % 16 == 0) return 16;
  if (n_inputs % 4 == 0 && a % 4 == 0) return 4;
  return 1;
}

PassAConfig default_pass_a_config(int vec, int64_t row_bytes, int64_t n_blocks, int block_len, bool lane_table,
                                  int n_cu) {
  const int64_t cg = row_bytes / vec;
  // Wide rows whose 4-block tasks (512-lane workgroups) fill one round of
  // the CUs: hold every block's sums and store them at the end of the task,
  // so the call reads, then writes (CHIME M = 256: 349 against 359 us).
  // With two or three blocks per task, or several rounds, the stores meet
  // the reads again and the per-block variants below are faster.
  if (lane_table && vec == 16 && cg >= 512 && n_cu > 0) {
    const int64_t units = n_blocks * ((cg + 511) / 512);
    if ((units + 3) / 4 <= n_cu && units > 3 * (int64_t)n_cu) {
      PassAConfig c;
      c.vec = vec;
      c.lpr = 512;
      c.variant = 4;
      c.grid = (int)((units + 3) / 4);
      return c;
    }
  }
  // Wide rows with at least one task per CU take the lane-replicated table
  // (no bank conflicts on the power lookups), measured fastest on MI355X:
  //  * >= 512 groups of 16 inputs: packed entries (one add per sample for
  //    both sums) in 1024-lane workgroups, one per CU, each streaming whole
  //    rows of a block (rows of 8 KiB: 316 us for 2 GiB at M = 1024 against
  //    333 us for the next best; equal at M = 256);
  //  * >= 256 groups: one row phase of 256 lanes, packed entries.
  if (lane_table && vec == 16 && cg >= 512 && n_blocks * ((cg + 1023) / 1024) >= 256) {
    const int64_t tasks = n_blocks * ((cg + 1023) / 1024);
    PassAConfig c;
    c.vec = vec;
    c.lpr = 1024;
    c.variant = 2;
    c.grid = (int)(tasks < (1 << 30) ? tasks : (1 << 30));
    return c;
  }
  if (lane_table && vec == 16 && cg >= 256 && n_blocks * ((cg + 255) / 256) >= 256) {
    const int64_t tasks = n_blocks * ((cg + 255) / 256);
    PassAConfig c;
    c.vec = vec;
    c.lpr = 256;
    c.variant = 1;    // packed entries: 2048-input serving frames 68.6 against 76.2 us unpacked
    c.grid = (int)(tasks < (1 << 30) ? tasks : (1 << 30));
    return c;
  }
  // Narrow rows with at least one task per CU: blocks side by side in
  // 256-lane workgroups with the packed table, every lane summing whole rows
  // (the Pathfinder shape: 53 against 57 us with row phases).
  if (lane_table && vec == 16 && cg < 256) {
    int lpb = 1;
    while (lpb < cg) lpb *= 2;
    const int64_t tasks = (n_blocks + 256 / lpb - 1) / (256 / lpb);
    if (tasks >= 256) {
      PassAConfig c;
      c.vec = vec;
      c.lpr = lpb;
      c.variant = 3;
      c.grid = (int)(tasks < (1 << 30) ? tasks : (1 << 30));
      return c;
    }
  }
  int lpr = 1;
  while (lpr < 256 && lpr < cg) lpr *= 2;
  // Keep at least ~2048 workgroups in flight: trade lanes per row for row
  // phases (reduced in LDS), down to 64 lanes, then on to 16 while a
  // workgroup's row phases do not outnumber the block's rows (the 256-input
  // serving frame, 192 blocks of 1 KiB rows: 17.1 against 28.0 us at 64).
  while (lpr > 64 && n_blocks * ((cg + lpr - 1) / lpr) < 2048) lpr /= 2;
  while (lpr > 16 && 512 / lpr <= block_len && n_blocks * ((cg + lpr - 1) / lpr) < 2048) lpr /= 2;
  const int64_t tasks = n_blocks * ((cg + lpr - 1) / lpr);
  PassAConfig c;
  c.vec = vec;
  c.lpr = lpr;
  c.variant = 0;
  c.grid = (int)(tasks < (1 << 30) ? (tasks > 0 ? tasks : 1) : (1 << 30));
  return c;
}

int launch_pass_a(const PassATask& t, const PassAConfig& c, hipStream_t s, PassEvents ev) {
  if (t.n_tasks <= 0) return SK_OK;
  const int grid = (int)(c.grid < t.n_tasks ? c.grid : t.n_tasks);
  switch (c.vec) {
    case 16: return launch_vec<16>(t, c.lpr, c.variant, grid, s, ev);
    case 4: return launch_vec<4>(t, c.lpr, c.variant, grid, s, ev);
    case 1: return launch_vec<1>(t, c.lpr, c.variant, grid, s, ev);
  }
  set_error("pass A: unsupported vector width %d", c.vec);
  return SK_ERR_INVALID_ARG;
}

}  // namespace sk
