// Pass A device code shared by the single-plan and batched kernels:
// decode, power table, and the per-lane row walk (Eq. singlesums).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sk_internal.h"
#include "sk_wave_dev.h"

namespace sk {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Power of one offset-encoded byte: high nibble = Re + 8, low = Im + 8.
__device__ __forceinline__ uint32_t code_power(uint32_t c) {
  const int re = (int)(c >> 4) - 8;
  const int im = (int)(c & 15u) - 8;
  return (uint32_t)(re * re + im * im);
}

#define SK_GLOBAL __attribute__((address_space(1)))

// Input rows always live in device (global) memory. Loading through a
// global-address-space pointer keeps the loads global_load_* even where the
// compiler cannot infer the address space (flat loads would also count
// against the LDS wait counter and serialise the table reads behind them).
template <int VEC>
struct Row {
  static constexpr int DW = VEC >= 4 ? VEC / 4 : 1;
  uint32_t w[DW];
  __device__ __forceinline__ void load(const uint8_t* p) {
    if constexpr (VEC == 16) {
      const u32x4 v = __builtin_nontemporal_load((const SK_GLOBAL u32x4*)p);
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else if constexpr (VEC == 4) {
      w[0] = __builtin_nontemporal_load((const SK_GLOBAL uint32_t*)p);
    } else {
      w[0] = *(const SK_GLOBAL uint8_t*)p;
    }
  }
  __device__ __forceinline__ uint32_t byte(int k) const {
    return (w[k >> 2] >> (8 * (k & 3))) & 0xFFu;
  }
};

template <int VEC>
__device__ __forceinline__ void accumulate_pair(const Row<VEC>& r0, const Row<VEC>& r1,
                                                const uint16_t* lut, uint32_t* s1, uint32_t* s2) {
  const u16x2 ones = {1, 1};
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    const uint32_t pp = (uint32_t)lut[r0.byte(k)] | ((uint32_t)lut[r1.byte(k)] << 16);
    const u16x2 P = __builtin_bit_cast(u16x2, pp);
    s2[k] = __builtin_amdgcn_udot2(P, P, s2[k], false);
    s1[k] = __builtin_amdgcn_udot2(P, ones, s1[k], false);
  }
}

template <int VEC>
__device__ __forceinline__ void accumulate_one(const Row<VEC>& r0, const uint16_t* lut,
                                               uint32_t* s1, uint32_t* s2) {
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    const uint32_t p = lut[r0.byte(k)];
    s1[k] += p;
    s2[k] += p * p;
  }
}

// Packed power table replicated per lane: the entry of code c for lane l is
// the dword at byte (c << 8) | (l % 64) * 4, 64 KiB in all, holding
// p | p^2 << 12 for code c. The 64 lanes of a wavefront always read 64
// distinct consecutive dwords (no bank conflicts whatever the codes), and
// one v_perm_b32 forms the address: byte 1 = the code byte, byte 0 = the
// lane's offset. Over at most 16 rows, sum p <= 2048 stays in
// the low 12 bits and sum p^2 <= 2^18 in the next 19, so one 32-bit add per
// sample (v_add3_u32 folds two rows) accumulates both sums; every 16 rows
// the packed sums are split into S1 and S2.
struct LanePackedLut {
  const uint8_t* base;
  uint32_t laneoff;
  __device__ __forceinline__ uint32_t at(uint32_t w, int k) const {
    const uint32_t sel = 0x0C0C0000u | ((uint32_t)(4 + k) << 8);
    return *reinterpret_cast<const uint32_t*>(base + __builtin_amdgcn_perm(w, laneoff, sel));
  }
};
constexpr int PACK_ROWS = 16;
constexpr int PACK_SHIFT = 12;

constexpr int LANE_LUT_DWORDS = 256 * 64;

template <int WG>
__device__ __forceinline__ void fill_lane_packed_lut(uint32_t* t, int tid) {
  for (int k = tid; k < LANE_LUT_DWORDS / 4; k += WG) {
    const uint32_t p = code_power((uint32_t)(k >> 4));
    const uint32_t e = p | (p * p << PACK_SHIFT);
    reinterpret_cast<u32x4*>(t)[k] = u32x4{e, e, e, e};
  }
}

// Batches of PHASE_ROWS rows of one lane's 16 columns, rows ph, ph + RP, ...
// of a batch that starts at the uniform pointer `p`. Four rows: two buffers of
// eight and the sums do not fit 128 registers. The 16 bytes may start anywhere
// (one global_load_dwordx4 either way).
constexpr int PHASE_ROWS = 4;
typedef u32x4 u32x4_any __attribute__((aligned(1)));

__device__ __forceinline__ u32x4 load16_any(const uint8_t* row, uint32_t off) {
  return __builtin_nontemporal_load((const SK_GLOBAL u32x4_any*)((const SK_GLOBAL uint8_t*)row + off));
}

// A whole batch: `off` = ph G + column, the row a scalar step.
template <int RP>
__device__ __forceinline__ void phased_load(u32x4 (&q)[PHASE_ROWS], const uint8_t* p, int64_t G, uint32_t off) {
#pragma unroll
  for (int u = 0; u < PHASE_ROWS; ++u) {
    // The row pointer in scalar registers and the lane's 32-bit offset in one
    // vector register: left to itself the compiler carries a 64-bit vector
    // address per row through the loop.
    const uint8_t* row = p + (int64_t)(u * RP) * G;
    asm("" : "+s"(row), "+v"(off));
    q[u] = load16_any(row, off);
  }
}

// Row r of a batch `left` rows before the block ends, and where it is read from: a
// row past the end reads the last one in its place, from column `past` on. (On the
// host too, where a test follows every address.)
__host__ __device__ __forceinline__ int phased_end_row(int r, int left) { return r < left ? r : left - 1; }
__host__ __device__ __forceinline__ uint32_t phased_end_col(int r, int left, uint32_t col, uint32_t past) {
  return r < left ? col : past;
}

// Where batch k of the last ones of a block is fetched, `left` rows before its end:
// row `at` on, of which `rows` are the block's, from column `col`. A batch past the
// end reads the last row, and from `past` in every lane: `col0` suits a lane's own
// rows, and the last row need not start where they do within a dword.
struct PhasedFetch {
  int at, rows;
  uint32_t col;
};
__host__ __device__ __forceinline__ PhasedFetch phased_fetch(int k, int step, int left, uint32_t col0, uint32_t past) {
  const bool any = k * step < left;
  const int at = any ? k * step : left - 1;
  return PhasedFetch{at, left - at, any ? col0 : past};
}

// A batch `left` rows before the block ends (phased_mask clears the rows past it).
// Row offsets are 24-bit products: the row index is below PHASE_ROWS RP and G below 2^24.
template <int RP>
__device__ __forceinline__ void phased_load_end(u32x4 (&q)[PHASE_ROWS], const uint8_t* p, int left, uint32_t G, int ph,
                                                uint32_t col, uint32_t past) {
  asm("" : "+v"(ph));   // offsets formed here, not kept from the first batch
#pragma unroll
  for (int u = 0; u < PHASE_ROWS; ++u) {
    const int r = ph + u * RP;
    q[u] = load16_any(p, __umul24((uint32_t)phased_end_row(r, left), G) + phased_end_col(r, left, col, past));
  }
}

// Rows past the end get the code of zero power (0x88: Re = Im = 0).
template <int RP>
__device__ __forceinline__ void phased_mask(u32x4 (&q)[PHASE_ROWS], int left, int ph) {
#pragma unroll
  for (int u = 0; u < PHASE_ROWS; ++u)
    if (ph + u * RP >= left) q[u] = u32x4{0x88888888u, 0x88888888u, 0x88888888u, 0x88888888u};
}

__device__ __forceinline__ void phased_add(const u32x4 (&q)[PHASE_ROWS], const LanePackedLut& lut, uint32_t (&acc)[16]) {
#pragma unroll
  for (int u = 0; u < PHASE_ROWS; u += 2)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        acc[4 * w + k] = acc[4 * w + k] + lut.at(q[u][w], k) + lut.at(q[u + 1][w], k);
      if (w & 1) __builtin_amdgcn_sched_barrier(0);   // 16 table reads in flight at most: more spill
    }
}

// Clears the counters in which the call's window kernel counts its finished slices:
// `clear` behind a kernel's last stores (ahead of its loads, the first rows' wait covers
// the store too: 0.5 us of pass A, 2048 inputs, 403 MB). The arguments are taken while
// they are still in the scalar cache and kept in registers: at the end of a long kernel
// they would come from host memory again (1 us of pass A, 2048 inputs, 2 GiB).
template <int WG>
struct CountsToClear {
  uint32_t* done;
  int32_t n, grid;
  __device__ __forceinline__ explicit CountsToClear(const PassATask& t)
      : done(t.done), n(t.n_done), grid((int32_t)gridDim.x) {
    asm volatile("" : "+s"(done), "+s"(n), "+s"(grid));
  }
  __device__ __forceinline__ void clear(int tid) const {
    if (n > 0)
      for (int64_t k = (int64_t)blockIdx.x * WG + tid; k < n; k += (int64_t)grid * WG) done[k] = 0u;
  }
};

// Nothing between packed runs.
struct NoBalance {
  __device__ __forceinline__ void operator()() {}
};

// Wavefronts that share a SIMD do not progress alike: the instruction
// arbiter favours the older one, so with equal work the younger one ends
// last and then runs alone, with half the loads in flight, for the end of
// the kernel (CHIME M = 256, variant 4: the first wavefront of each SIMD
// ended its reads about 55 us before the second). After every packed run a
// wavefront posts its progress in LDS and compares it with its partner's
// (another wavefront of the workgroup on the same SIMD): ahead, it drops to
// priority 0; level or behind, it takes priority 2. No wavefront waits.
struct SimdBalance {
  uint32_t* prog;   // LDS, one word per wavefront of the workgroup
  int self, partner;
  uint32_t done;
  __device__ __forceinline__ void operator()() {
    ++done;
    // Every lane stores the same value: no divergent branch.
    __atomic_store_n(&prog[self], done, __ATOMIC_RELAXED);
    const uint32_t other = __builtin_amdgcn_readfirstlane(__atomic_load_n(&prog[partner], __ATOMIC_RELAXED));
    // One asm block for the compare and both priorities, so the compiler's
    // control flow (and its register allocation) is not split.
    asm volatile("s_cmp_gt_u32 %0, %1\n\ts_cbranch_scc0 1f\n\ts_setprio 0\n\ts_branch 2f\n1:\n\ts_setprio 2\n2:"
                 :: "s"(__builtin_amdgcn_readfirstlane(done)), "s"(other) : "scc");
  }
};

// SIMD of the calling wavefront (HW_ID bits 5:4).
__device__ __forceinline__ uint32_t simd_id() {
  return (uint32_t)__builtin_amdgcn_s_getreg(4 | (4 << 6) | (1 << 11));
}

// First half of setting up SimdBalance for a workgroup of `waves`
// wavefronts: each posts its SIMD and zero progress. The caller then
// synchronises the workgroup before simd_balance_pair.
__device__ __forceinline__ void simd_balance_post(uint32_t* sid, uint32_t* prog, int tid) {
  if ((tid & 63) == 0) {
    sid[tid >> 6] = simd_id();
    prog[tid >> 6] = 0;
  }
}

// Second half: the partner is the first other wavefront on the same SIMD
// (none: the wavefront is its own partner and always takes priority 2).
__device__ __forceinline__ SimdBalance simd_balance_pair(const uint32_t* sid, uint32_t* prog, int waves) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int partner = w;
  for (int j = waves - 1; j >= 0; --j)
    if (j != w && sid[j] == sid[w]) partner = j;
  return SimdBalance{prog, w, __builtin_amdgcn_readfirstlane(partner), 0u};
}

// Rows ph, ph + RP, ... (< M) of this lane with the packed table, in loads of
// U rows, unpacking every PACK_ROWS rows; `bal` runs after every packed run.
template <int VEC, int RP, int U, typename Balance = NoBalance>
__device__ __forceinline__ void sum_rows_packed(const uint8_t* base, int64_t G, int M, int ph,
                                                const LanePackedLut& lut, uint32_t* s1, uint32_t* s2,
                                                Balance&& bal = Balance()) {
  static_assert(VEC >= 4 && U % 2 == 0 && PACK_ROWS % U == 0, "whole row pairs per packed run");
  const int nrow = ph < M ? (M - ph + RP - 1) / RP : 0;
  const int64_t step = (int64_t)RP * G;
  const uint8_t* p = base + (int64_t)ph * G;
  for (int done = 0; done < nrow; done += PACK_ROWS) {
    const int n = nrow - done < PACK_ROWS ? nrow - done : PACK_ROWS;
    uint32_t acc[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) acc[k] = 0;
    int r = 0;
    for (; r + U <= n; r += U) {
      Row<VEC> q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) q[u].load(p + u * step);
      p += U * step;
#pragma unroll
      for (int u = 0; u < U; u += 2)
#pragma unroll
        for (int k = 0; k < VEC; ++k)
          acc[k] = acc[k] + lut.at(q[u].w[k >> 2], k & 3) + lut.at(q[u + 1].w[k >> 2], k & 3);
    }
    for (; r < n; ++r) {
      Row<VEC> q;
      q.load(p);
      p += step;
#pragma unroll
      for (int k = 0; k < VEC; ++k) acc[k] += lut.at(q.w[k >> 2], k & 3);
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      s1[k] += acc[k] & ((1u << PACK_SHIFT) - 1);
      s2[k] += acc[k] >> PACK_SHIFT;
    }
    bal();
  }
}

// Rows of this lane in batches of U: r = ph, ph + RP, ... (< M), the loads
// of a batch issued together, then reduced in row pairs.
template <int VEC, int RP, int U>
__device__ __forceinline__ void sum_rows(const uint8_t* base, int64_t G, int M, int ph,
                                         const uint16_t* lut, uint32_t* s1, uint32_t* s2) {
  const int nrow = ph < M ? (M - ph + RP - 1) / RP : 0;
  const int nb = nrow / U;
  int r = ph;
  for (int bt = 0; bt < nb; ++bt) {
    Row<VEC> q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u].load(base + (int64_t)(r + u * RP) * G);
#pragma unroll
    for (int u = 0; u < U / 2; ++u) accumulate_pair<VEC>(q[2 * u], q[2 * u + 1], lut, s1, s2);
    r += U * RP;
  }
  for (; r + RP < M; r += 2 * RP) {
    Row<VEC> q0, q1;
    q0.load(base + (int64_t)r * G);
    q1.load(base + (int64_t)(r + RP) * G);
    accumulate_pair<VEC>(q0, q1, lut, s1, s2);
  }
  if (r < M) {
    Row<VEC> q0;
    q0.load(base + (int64_t)r * G);
    accumulate_one<VEC>(q0, lut, s1, s2);
  }
}

// One 256-lane task with the packed lane table (Eq. singlesums), every lane
// (tid, 0..255) summing whole rows of one (block, column group). lpb = lanes per block row:
// 256 for wide rows (task = t.blocks_per_task consecutive blocks, walked one
// after the other, of a chunk of 256 column groups); a power of two >= the
// row's column groups otherwise (task = t.blocks_per_task = 256 / lpb
// consecutive blocks side by side, lane l on block l / lpb, column group
// l % lpb). Needs the PassATask fields chunks, blocks_per_task, block0 and
// block_end set to match. With wide rows and t.cs set, the task also writes
// its blocks' S1 total (the chunk sum of pass B chunks of blocks_per_task
// blocks); narrow rows need t.cs null.
template <int U, typename Balance = NoBalance>
__device__ __forceinline__ void pass_a_task_side_by_side(const PassATask& t, int lpb, int64_t task,
                                                         const LanePackedLut& lut, int tid,
                                                         Balance&& bal = Balance()) {
  constexpr int VEC = 16;
  const int64_t bg = task / t.chunks;
  const int ch = (int)(task % t.chunks);
  int64_t b, b_end;
  int g;
  if (lpb >= 256) {
    b = t.block0 + bg * t.blocks_per_task;
    b_end = b + t.blocks_per_task;
    g = ch * 256 + tid;
  } else {
    b = t.block0 + bg * t.blocks_per_task + tid / lpb;
    b_end = b + 1;
    g = tid % lpb;
  }
  if (b_end > t.block_end) b_end = t.block_end;
  if (g >= t.col_groups) return;
  const int M = t.block_len;
  const int64_t G = t.row_bytes;
  const int N = t.n_inputs, B = t.n_blocks;
  const int64_t col = (int64_t)g * VEC;
  const int64_t f = col / N, i = col % N;
  const int64_t b_first = b;
  uint32_t c[VEC];
#pragma unroll
  for (int k = 0; k < VEC; ++k) c[k] = 0;
  for (; b < b_end; ++b) {
    uint32_t s1[VEC], s2[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) s1[k] = s2[k] = 0;
    sum_rows_packed<VEC, 1, U>(t.x + b * M * G + (int64_t)g * VEC, G, M, 0, lut, s1, s2, bal);
    int32_t* d1 = t.s1 + (f * B + b) * N + i;
    int32_t* d2 = t.s2 + (f * B + b) * N + i;
#pragma unroll
    for (int k = 0; k < VEC; k += 4) {
      *reinterpret_cast<u32x4*>(d1 + k) = u32x4{s1[k], s1[k + 1], s1[k + 2], s1[k + 3]};
      *reinterpret_cast<u32x4*>(d2 + k) = u32x4{s2[k], s2[k + 1], s2[k + 2], s2[k + 3]};
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) c[k] += s1[k];
  }
  if (lpb >= 256 && t.cs) {
    // S1 over the task's blocks (wide rows): the chunk sums the prefix scan
    // reads instead of the rows when the task's blocks are one pass B chunk.
    const int Q = t.blocks_per_task;
    const int64_t nk = (t.n_blocks + Q - 1) / Q;
    int32_t* d = t.cs + (f * nk + (b_first - t.block0) / Q) * N + i;
#pragma unroll
    for (int k = 0; k < VEC; k += 4) *reinterpret_cast<u32x4*>(d + k) = u32x4{c[k], c[k + 1], c[k + 2], c[k + 3]};
  }
}

// One 512-lane task of Q consecutive blocks over 512 column groups (chunk
// task % chunks), every lane summing whole rows of one column group, with
// all Q blocks' sums held in registers and stored after the last block, so
// the stores do not interleave with the task's reads; with t.cs set, the S1
// total of the Q blocks too (the chunk sums of pass B chunks of Q blocks).
// Contains no barrier.
template <int Q, int U, typename Balance>
__device__ __forceinline__ void pass_a_task_deferred(const PassATask& t, int64_t task, const LanePackedLut& lut,
                                                     Balance&& bal) {
  constexpr int VEC = 16;
  const int tid = threadIdx.x;
  const int b0 = t.block0 + (int)(task / t.chunks) * Q;
  const int g = (int)(task % t.chunks) * 512 + tid;
  if (g >= t.col_groups) return;
  const int M = t.block_len, N = t.n_inputs, B = t.n_blocks;
  const int64_t G = t.row_bytes;
  uint32_t a1[Q][VEC], a2[Q][VEC];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
#pragma unroll
    for (int k = 0; k < VEC; ++k) a1[q][k] = a2[q][k] = 0;
    if (b0 + q < t.block_end)
      sum_rows_packed<VEC, 1, U>(t.x + (int64_t)(b0 + q) * M * G + (int64_t)g * VEC, G, M, 0, lut, a1[q], a2[q], bal);
  }
  __builtin_amdgcn_s_setprio(0);
  const int64_t col = (int64_t)g * VEC;
  const int64_t f = col / N, i = col % N;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (b0 + q >= t.block_end) continue;
    int32_t* d1 = t.s1 + (f * B + b0 + q) * N + i;
    int32_t* d2 = t.s2 + (f * B + b0 + q) * N + i;
#pragma unroll
    for (int k = 0; k < VEC; k += 4) {
      *reinterpret_cast<u32x4*>(d1 + k) = u32x4{a1[q][k], a1[q][k + 1], a1[q][k + 2], a1[q][k + 3]};
      *reinterpret_cast<u32x4*>(d2 + k) = u32x4{a2[q][k], a2[q][k + 1], a2[q][k + 2], a2[q][k + 3]};
    }
  }
  if (t.cs) {
    const int64_t nk = (t.n_blocks + Q - 1) / Q;
    int32_t* d = t.cs + (f * nk + (b0 - t.block0) / Q) * N + i;
#pragma unroll
    for (int k = 0; k < VEC; k += 4) {
      u32x4 c = {a1[0][k], a1[0][k + 1], a1[0][k + 2], a1[0][k + 3]};
#pragma unroll
      for (int q = 1; q < Q; ++q) c += u32x4{a1[q][k], a1[q][k + 1], a1[q][k + 2], a1[q][k + 3]};
      *reinterpret_cast<u32x4*>(d + k) = c;
    }
  }
}

// Stores four columns from column c on (S1 a, S2 b) of block `blk`; they may
// straddle channels or pass the row's end, and the sums' rows need only 4-byte
// alignment.
__device__ __forceinline__ void store_quad(const PassATask& t, int blk, int c, u32x4 a, u32x4 b) {
  typedef u32x4 u32x4_word __attribute__((aligned(4)));
  const int N = t.n_inputs, B = t.n_blocks;
  int f = c / N, i = c - f * N;
  const int64_t d = ((int64_t)f * B + blk) * N + i;
  if (i + 4 <= N) {
    *reinterpret_cast<u32x4_word*>(t.s1 + d) = a;
    *reinterpret_cast<u32x4_word*>(t.s2 + d) = b;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (c + j >= t.row_bytes) break;
      const int64_t e = ((int64_t)f * B + blk) * N + i;
      t.s1[e] = (int32_t)a[j];
      t.s2[e] = (int32_t)b[j];
      if (++i == N) {
        i = 0;
        ++f;
      }
    }
  }
}

// Sums (S1 in v[0 .. 15], S2 in v[16 .. 31]) of rows ph, ph + RP, ... < M of this
// lane's 16 columns, `col0` from the uniform pointer p on; `past` is where a load
// past the last row goes. prepare() runs with the first rows in flight and leaves
// the table filled.
template <int RP, typename Prepare>
__device__ __forceinline__ void phased_sums(const uint8_t* p, int G, int M, int ph, uint32_t col0, uint32_t past,
                                            const LanePackedLut& lut, uint32_t (&v)[32], Prepare&& prepare) {
  constexpr int VEC = 16, STEP = PHASE_ROWS * RP;   // rows of the block per batch
  const int64_t step_bytes = (int64_t)STEP * G;
  u32x4 qa[PHASE_ROWS], qb[PHASE_ROWS];
  phased_load_end<RP>(qa, p, M, G, ph, col0, past);
  prepare();
  uint32_t acc[VEC];
#pragma unroll
  for (int k = 0; k < 2 * VEC; ++k) v[k] = 0;
#pragma unroll
  for (int k = 0; k < VEC; ++k) acc[k] = 0;
  const auto unpack = [&] {
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      v[k] += acc[k] & ((1u << PACK_SHIFT) - 1);
      v[VEC + k] += acc[k] >> PACK_SHIFT;
      acc[k] = 0;
    }
  };
  const uint32_t off = __umul24(ph, G) + col0;
  int left = M;
  // Whole batches four at a time (16 rows, one packed run), the next one in
  // flight, while another whole batch follows them; then the at most five
  // batches that remain (20 rows still fit the packed sums: 20 * 128 < 2^12).
  for (; left >= 5 * STEP; left -= 4 * STEP) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      p += step_bytes;
      phased_load<RP>(qb, p, G, off);
      phased_add(qa, lut, acc);
      p += step_bytes;
      phased_load<RP>(qa, p, G, off);
      phased_add(qb, lut, acc);
    }
    unpack();
  }
  // (A fetch past the end reads the last row: under a branch instead, the wait
  // for the batch before it would cover the fetch too.)
  const auto fetch = [&](u32x4(&q)[PHASE_ROWS], int k) {
    const PhasedFetch f = phased_fetch(k, STEP, left, col0, past);
    phased_load_end<RP>(q, p + (int64_t)f.at * G, f.rows, G, ph, f.col, past);
  };
  const auto take = [&](u32x4(&q)[PHASE_ROWS], int k) {
    phased_mask<RP>(q, left - k * STEP, ph);
    phased_add(q, lut, acc);
  };
  fetch(qb, 1);
  take(qa, 0);
  if (left > STEP) {
    fetch(qa, 2);
    take(qb, 1);
    if (left > 2 * STEP) {
      fetch(qb, 3);
      take(qa, 2);
      if (left > 3 * STEP) {
        fetch(qa, 4);
        take(qb, 3);
        if (left > 4 * STEP) take(qa, 4);
      }
    }
  }
  unpack();
}

// Task of this workgroup. by_xcd: consecutive tasks on one XCD (workgroups go round
// the eight), so a line that two tasks share is fetched into one L2.
__device__ __forceinline__ int pass_a_task_of(const PassATask& t) {
  const int id = blockIdx.x, n = gridDim.x;
  if (!t.by_xcd) return id;
  const int q = n >> 3, r = n & 7, x = id & 7;
  return x * q + (x < r ? x : r) + (id >> 3);
}

// Accumulator row stride of pass_a_task_phased: S1 of column k of unit g lies at
// k S + g of `red`, S2 at (16 + k) S + g (32 S words).
__host__ __device__ constexpr int phased_stride(int lpr) { return lpr + 1; }

// Column a lane of unit u reads from, from the block of unit u0 on (on the host too,
// as above).
__host__ __device__ __forceinline__ uint32_t phased_column(int u, int u0, int M, int G, int cg, int units) {
  const int w = u < units ? u : units - 1, bl = w / cg, c = (w - bl * cg) * 16;
  return (uint32_t)(bl - u0 / cg) * (uint32_t)M * (uint32_t)G + (uint32_t)(c < G - 16 ? c : G - 16);
}

// One task of row phases on a 512-lane workgroup (see pass_a_phased_kernel):
// units u0 .. u0 + LPR - 1 times 512 / LPR phases. prepare() runs with the first
// rows in flight and leaves the table filled; red holds zeros then, or, with
// OVER, is cleared here once the table is no longer needed. AGAIN: red holds
// zeros again at the end (the caller's next barrier makes them seen).
template <int LPR, bool OVER, bool AGAIN, typename Prepare>
__device__ __forceinline__ void pass_a_task_phased(const PassATask& t, int u0, const LanePackedLut& lut, uint32_t* red,
                                                   int tid, Prepare&& prepare) {
  static_assert(LPR >= 16, "a row of 16 lanes holds the units of one or more row groups");
  constexpr int VEC = 16, RP = 512 / LPR;
  constexpr int S = phased_stride(LPR);
  constexpr int NV = LPR >= 64 ? 32 : LPR == 32 ? 16 : 8;   // sums a lane adds
  const int lc = tid % LPR;
  const int M = t.block_len, ph = tid / LPR;
  const int G = (int)t.row_bytes, cg = t.col_groups;
  const int units = t.n_blocks * cg;
  const int b_first = u0 / cg;            // uniform: the lanes' offsets start at this block
  const uint32_t col0 = phased_column(u0 + lc, u0, M, G, cg, units);
  uint32_t v[2 * VEC];
  phased_sums<RP>(t.x + (int64_t)b_first * M * G, G, M, ph, col0, col0, lut, v, prepare);
  if constexpr (RP == 1) {
    const int u = u0 + lc;
    if (u < units) {
      const int blk = u / cg, c = (u - blk * cg) * VEC, c0 = c < G - VEC ? c : G - VEC;
#pragma unroll
      for (int k = 0; k < VEC; k += 4)
        store_quad(t, blk, c0 + k, u32x4{v[k], v[k + 1], v[k + 2], v[k + 3]},
                   u32x4{v[VEC + k], v[VEC + k + 1], v[VEC + k + 2], v[VEC + k + 3]});
    }
    return;
  }
  if constexpr (OVER) {
    lds_barrier();
    for (int o = tid; o < 2 * VEC * S; o += 512) red[o] = 0u;
    lds_barrier();
  }
  // Sum over the wavefront's row groups, then over the wavefronts.
  const int lane = tid & 63;
  if constexpr (LPR >= 64) {
#pragma unroll
    for (int k = 0; k < NV; ++k) atomicAdd(&red[k * S + lc], v[k]);
  } else {
    uint32_t c[VEC];
#pragma unroll
    for (int m = 0; m < VEC; ++m) {
      swap_halves(v[2 * m], v[2 * m + 1]);
      c[m] = v[2 * m] + v[2 * m + 1];
    }
    if constexpr (LPR == 32) {
#pragma unroll
      for (int m = 0; m < VEC; ++m) atomicAdd(&red[(2 * m + (lane >> 5)) * S + lc], c[m]);
    } else {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        swap_rows(c[2 * q], c[2 * q + 1]);
        const uint32_t x = c[2 * q] + c[2 * q + 1];
        atomicAdd(&red[wave_value_of_row(q, lane >> 4) * S + lc], x);
      }
    }
  }
  lds_barrier();
  for (int o = tid; o < 4 * LPR; o += 512) {
    const int lg = o >> 2, k = (o & 3) * 4, u = u0 + lg;
    if (u < units) {
      const int blk = u / cg, c = (u - blk * cg) * VEC, c0 = c < G - VEC ? c : G - VEC;
      const uint32_t* r1 = red + k * S + lg;
      const uint32_t* r2 = r1 + VEC * S;
      store_quad(t, blk, c0 + k, u32x4{r1[0], r1[S], r1[2 * S], r1[3 * S]}, u32x4{r2[0], r2[S], r2[2 * S], r2[3 * S]});
    }
    if constexpr (AGAIN)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[(k + j) * S + lg] = red[(VEC + k + j) * S + lg] = 0u;
  }
}

// Accumulator row stride of pass_a_task_shifted: column q of unit g at q S + g of
// `red` (S1; S2 at (16 + q) S + g), 32 S words. 128 units take no pad: two workgroups
// with table and sums just fill a CU's LDS.
__host__ __device__ constexpr int shifted_stride(int lpr) { return lpr < 128 ? lpr + 1 : lpr; }

// What a lane of pass_a_task_shifted reads (on the host too, as above): its unit
// `lc` of the task's, its row phase, its unit's block and first column, and the
// columns its loads start at, from 4 bytes before the task's first block on.
struct ShiftedLane {
  int lc, ph, blk, c16, shift, c;   // c: first column of the lane's windows
  bool live;
  uint32_t col0, past;
};
template <int LPR>
__host__ __device__ __forceinline__ ShiftedLane shifted_lane(uintptr_t x, int u0, int tid, int M, int G, int cg, int units) {
  constexpr int VEC = 16;
  // A wavefront takes UW units and 64 / UW phases that are equal mod 4: one shift a unit.
  constexpr int UW = LPR <= 32 ? 16 : LPR / 2;
  const int lane = tid & 63, wave = tid >> 6;
  ShiftedLane l;
  l.lc = (LPR > UW ? (wave >> 2) * UW : 0) + lane % UW;
  l.ph = (wave & 3) + 4 * (lane / UW + (LPR > UW ? 0 : (wave >> 2) * (64 / UW)));
  l.live = u0 + l.lc < units;
  const int u = l.live ? u0 + l.lc : units - 1;
  l.blk = u / cg;
  l.c16 = (u - l.blk * cg) * VEC;
  // Bytes from an aligned dword to the lane's first row; its rows' windows start
  // that many columns before the unit, or as far on as the row's end allows.
  l.shift = (int)(((uint32_t)x + ((uint32_t)l.blk * (uint32_t)M + (uint32_t)l.ph) * (uint32_t)G) & 3u);
  const int end = G - VEC + (-(l.shift + G - VEC) & 3);
  l.c = l.c16 - l.shift < end ? l.c16 - l.shift : end;
  // Offsets count from 4 bytes before the block: a window may start before its row.
  const uint32_t at = (uint32_t)(l.blk - u0 / cg) * (uint32_t)M * (uint32_t)G + 4u;
  l.col0 = at + (uint32_t)l.c;
  l.past = at + (uint32_t)(l.c < G - VEC ? l.c : G - VEC);
  return l;
}

// One task of shifted row phases on a 512-lane workgroup (see
// pass_a_shifted_kernel): units u0 .. u0 + LPR - 1, of which the last is only read
// for the columns it has of the one before. prepare() runs with the first rows in
// flight and ends with a barrier behind which the table is filled and red holds
// zeros; red holds zeros again at the end (the next barrier makes them seen).
template <int LPR, typename Prepare>
__device__ __forceinline__ void pass_a_task_shifted(const PassATask& t, int u0, const LanePackedLut& lut, uint32_t* red,
                                                    int tid, Prepare&& prepare) {
  constexpr int VEC = 16, RP = 512 / LPR, S = shifted_stride(LPR);
  static_assert(RP % 4 == 0, "a lane's rows lie a multiple of 4 bytes apart");
  constexpr int UW = LPR <= 32 ? 16 : LPR / 2;
  const int lane = tid & 63;
  const int M = t.block_len, G = (int)t.row_bytes, cg = t.col_groups;
  const int units = t.n_blocks * cg;
  const int b_first = u0 / cg;
  const ShiftedLane l = shifted_lane<LPR>(reinterpret_cast<uintptr_t>(t.x), u0, tid, M, G, cg, units);
  const int lc = l.lc, ph = l.ph, c16 = l.c16, s = l.shift, c = l.c;
  const bool live = l.live;
  const uint32_t col0 = l.col0, past = l.past;
  uint32_t v[2 * VEC];
  phased_sums<RP>(t.x + (int64_t)b_first * M * G - 4, G, M, ph, col0, past, lut, v, prepare);
  // Column c + k goes to place d = c + k - c16 of the unit (below 0: of the unit
  // before); what lies in another row, or is summed by the unit before, is left out.
  const int first = lc == 0 ? c16 : c16 - s > 0 ? c16 - s : 0;
  const int lo = first - c;
  const int hi = G - c < VEC ? G - c : VEC;
  const uint32_t n = live && hi > lo ? (uint32_t)(hi - lo) : 0u;
  const auto add = [&](int val, uint32_t x) {
    const int k = val & 15, d = c - c16 + k;
    if ((uint32_t)(k - lo) < n) atomicAdd(red + ((val & 16) + (d & 15)) * S + lc + (d >> 4), x);
  };
  if constexpr (UW == 64) {
#pragma unroll
    for (int k = 0; k < 2 * VEC; ++k) add(k, v[k]);
  } else {
    uint32_t x[VEC];
#pragma unroll
    for (int m = 0; m < VEC; ++m) {
      swap_halves(v[2 * m], v[2 * m + 1]);
      x[m] = v[2 * m] + v[2 * m + 1];
    }
    if constexpr (UW == 32) {
#pragma unroll
      for (int m = 0; m < VEC; ++m) add(2 * m + (lane >> 5), x[m]);
    } else {
#pragma unroll
      for (int q = 0; q < VEC / 2; ++q) {
        swap_rows(x[2 * q], x[2 * q + 1]);
        add(wave_value_of_row(q, lane >> 4), x[2 * q] + x[2 * q + 1]);
      }
    }
  }
  lds_barrier();
  for (int o = tid; o < 4 * LPR; o += 512) {
    const int lg = o >> 2, k = (o & 3) * 4, w = u0 + lg;
    uint32_t* r1 = red + k * S + lg;
    uint32_t* r2 = r1 + VEC * S;
    if (lg < LPR - 1 && w < units) {
      const int b = w / cg, col = (w - b * cg) * VEC + k;
      if (col < G)
        store_quad(t, b, col, u32x4{r1[0], r1[S], r1[2 * S], r1[3 * S]}, u32x4{r2[0], r2[S], r2[2 * S], r2[3 * S]});
    }
  }
}

}  // namespace sk
