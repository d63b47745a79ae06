// Wavefront sums (lane swaps and row rotations) and the LDS barrier, shared by
// pass A and pass B.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sk {

// Barrier that orders LDS alone: loads from global memory stay in flight
// across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------------------ wavefront sums
//
// One fixed tree for every value: lanes l and l + 32 first (v_permlane32_swap),
// then rows 0 + 1 and 2 + 3 of the result (v_permlane16_swap), then within a
// row of 16 lanes l + 8, l + 4, l + 2, l + 1 (DPP row rotations). Two values
// share each swap step (a reduce-scatter), so n values cost about n/4 of n
// separate reductions, and each value is added in the same order whichever
// values it is reduced with: results do not depend on the tile.

template <typename T>
__device__ __forceinline__ void swap_halves(T& x, T& y) {
  // After the swap, x holds x's lanes 0-31 and y's lanes 0-31 (in lanes
  // 32-63); y holds x's lanes 32-63 (in lanes 0-31) and y's lanes 32-63.
  if constexpr (sizeof(T) == 4) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                    false, false);
    x = __builtin_bit_cast(T, (uint32_t)r[0]);
    y = __builtin_bit_cast(T, (uint32_t)r[1]);
  } else {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    u2 a = __builtin_bit_cast(u2, x), b = __builtin_bit_cast(u2, y);
    const auto r0 = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
    const auto r1 = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
    a.x = r0[0]; b.x = r0[1];
    a.y = r1[0]; b.y = r1[1];
    x = __builtin_bit_cast(T, a);
    y = __builtin_bit_cast(T, b);
  }
}

template <typename T>
__device__ __forceinline__ void swap_rows(T& x, T& y) {
  // Rows of 16 lanes: x becomes (x0, y0, x2, y2), y becomes (x1, y1, x3, y3).
  if constexpr (sizeof(T) == 4) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                    false, false);
    x = __builtin_bit_cast(T, (uint32_t)r[0]);
    y = __builtin_bit_cast(T, (uint32_t)r[1]);
  } else {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    u2 a = __builtin_bit_cast(u2, x), b = __builtin_bit_cast(u2, y);
    const auto r0 = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
    const auto r1 = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    a.x = r0[0]; b.x = r0[1];
    a.y = r1[0]; b.y = r1[1];
    x = __builtin_bit_cast(T, a);
    y = __builtin_bit_cast(T, b);
  }
}

// Lane l + r (mod 16, within its row) of v, every row enabled.
template <int R, typename T>
__device__ __forceinline__ T row_rot(T v) {
  constexpr int CTRL = 0x120 + R;   // DPP row_ror:R
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
  } else {
    typedef int i2 __attribute__((ext_vector_type(2)));
    i2 a = __builtin_bit_cast(i2, v);
    a.x = __builtin_amdgcn_mov_dpp(a.x, CTRL, 0xF, 0xF, false);
    a.y = __builtin_amdgcn_mov_dpp(a.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(T, a);
  }
}

template <typename T>
__device__ __forceinline__ T row_total(T v) {
  v = v + row_rot<8>(v);
  v = v + row_rot<4>(v);
  v = v + row_rot<2>(v);
  v = v + row_rot<1>(v);
  return v;
}

// The same in 32 bits up to the last addition, which is in 64: sums whose halves
// fit (unsigned) need no wider steps before it.
__device__ __forceinline__ uint64_t row_total_wide(uint32_t v) {
  v = v + row_rot<8>(v);
  v = v + row_rot<4>(v);
  v = v + row_rot<2>(v);
  return (uint64_t)v + row_rot<1>(v);
}
__device__ __forceinline__ uint64_t row_total_wide(uint64_t v) { return row_total(v); }

// Integer sums of NV values (NV a power of two >= 2) over the wavefront, laid
// out as wave_sums.
template <int NV, typename T>
__device__ __forceinline__ void wave_sums_wide(const T (&v)[NV], uint64_t (&out)[(NV + 3) / 4]) {
  constexpr int NC = NV / 2;
  T c[NC];
#pragma unroll
  for (int m = 0; m < NC; ++m) {
    T x = v[2 * m], y = v[2 * m + 1];
    swap_halves(x, y);
    c[m] = x + y;
  }
#pragma unroll
  for (int q = 0; q < (NV + 3) / 4; ++q) {
    T x = c[2 * q], y = 2 * q + 1 < NC ? c[2 * q + 1] : c[2 * q];
    swap_rows(x, y);
    out[q] = row_total_wide(x + y);
  }
}

// Sums each of NV values (NV a power of two >= 2) over the wavefront.
// Value j ends in every lane of the row of out[j / 4] that
// wave_value_of_row names.
template <int NV, typename T>
__device__ __forceinline__ void wave_sums(const T (&v)[NV], T (&out)[(NV + 3) / 4]) {
  static_assert(NV >= 2 && (NV & (NV - 1)) == 0, "a power of two, at least 2");
  constexpr int NC = NV / 2;
  T c[NC];
#pragma unroll
  for (int m = 0; m < NC; ++m) {
    T x = v[2 * m], y = v[2 * m + 1];
    swap_halves(x, y);
    c[m] = x + y;
  }
#pragma unroll
  for (int q = 0; q < (NV + 3) / 4; ++q) {
    T x = c[2 * q], y = 2 * q + 1 < NC ? c[2 * q + 1] : c[2 * q];
    swap_rows(x, y);
    out[q] = row_total(x + y);
  }
}

// The value a lane of row r holds in out[q] after wave_sums: 4q + 2 (r & 1) + (r >> 1).
__device__ __forceinline__ int wave_value_of_row(int q, int r) { return 4 * q + 2 * (r & 1) + (r >> 1); }

}  // namespace sk
