// Walks the loads of pass A's row-phase kernels on the host, with the kernels' own
// address functions: every lane, every batch of rows (whole ones and the last ones,
// fetches past a block's end among them). One call per line of standard input:
// "5 | 6 | b, units per workgroup (0: the library's), N, F, M, blocks, address mod 4096";
// prints the lowest and highest byte read, counted from the frame's first, and the
// units per workgroup. Built with hipcc for the host alone.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "sk_internal.h"
#include "sk_pass_a_dev.h"

using namespace sk;

struct Range {
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  void load(int64_t at) {
    if (at < lo) lo = at;
    if (at + 15 > hi) hi = at + 15;
  }
};

// The loads of phased_sums: `base` is p's offset from the frame's first byte.
static void walk(Range& r, int rp, int64_t base, int64_t G, int M, int ph, uint32_t col0, uint32_t past) {
  const int step = PHASE_ROWS * rp;
  int left = M;
  const auto end = [&](int64_t p, int rows, uint32_t col) {
    for (int u = 0; u < PHASE_ROWS; ++u) {
      const int row = ph + u * rp;
      r.load(p + (int64_t)phased_end_row(row, rows) * G + phased_end_col(row, rows, col, past));
    }
  };
  end(base, M, col0);
  for (; left >= 5 * step; left -= 4 * step)
    for (int h = 0; h < 4; ++h) {
      base += step * G;
      for (int u = 0; u < PHASE_ROWS; ++u) r.load(base + (int64_t)(ph + u * rp) * G + col0);
    }
  for (int k = 1; k <= 4; ++k) {
    const PhasedFetch f = phased_fetch(k, step, left, col0, past);
    end(base + (int64_t)f.at * G, f.rows, f.col);
    if (left <= k * step) break;
  }
}

template <int LPR>
static void walk_phased(Range& r, int64_t task, int M, int G, int cg, int64_t units) {
  const int u0 = (int)task * LPR;
  for (int tid = 0; tid < 512; ++tid) {
    const uint32_t col = phased_column(u0 + tid % LPR, u0, M, G, cg, (int)units);
    walk(r, 512 / LPR, (int64_t)(u0 / cg) * M * G, G, M, tid / LPR, col, col);
  }
}

template <int LPR>
static void walk_shifted(Range& r, uintptr_t x, int64_t task, int M, int G, int cg, int64_t units) {
  const int u0 = (int)task * (LPR - 1);
  for (int tid = 0; tid < 512; ++tid) {
    const ShiftedLane l = shifted_lane<LPR>(x, u0, tid, M, G, cg, (int)units);
    walk(r, 512 / LPR, (int64_t)(u0 / cg) * M * G - 4, G, M, l.ph, l.col0, l.past);
  }
}

int main() {
  char kind;
  int lanes, N, F, M, B, at;
  while (scanf(" %c %d %d %d %d %d %d", &kind, &lanes, &N, &F, &M, &B, &at) == 7) {
    const int64_t G = (int64_t)N * F;
    const uint8_t* x = (const uint8_t*)(uintptr_t)(0x700000000000ull + at);
    const bool shifted = kind == '6';
    if (!lanes) lanes = shifted ? pass_a_shifted_lanes(x, G, B, M, 256) : pass_a_phased_lanes(x, G, N, B, M, 256);
    const int cg = (int)((G + (shifted ? 18 : 15)) / 16), stored = shifted ? lanes - 1 : lanes;
    const int64_t units = (int64_t)cg * B;
    Range r;
    if (stored > 0) {
      const int64_t tasks = (units + stored - 1) / stored;
      for (int64_t t = 0; t < tasks; ++t) {
        if (t >= 8 && t < tasks - 8) continue;   // the ends of the frame
        if (shifted) {
          switch (lanes) {
            case 16: walk_shifted<16>(r, (uintptr_t)x, t, M, (int)G, cg, units); break;
            case 32: walk_shifted<32>(r, (uintptr_t)x, t, M, (int)G, cg, units); break;
            case 64: walk_shifted<64>(r, (uintptr_t)x, t, M, (int)G, cg, units); break;
            case 128: walk_shifted<128>(r, (uintptr_t)x, t, M, (int)G, cg, units); break;
            default: return 2;
          }
        } else {
          switch (lanes) {
            case 16: walk_phased<16>(r, t, M, (int)G, cg, units); break;
            case 32: walk_phased<32>(r, t, M, (int)G, cg, units); break;
            case 64: walk_phased<64>(r, t, M, (int)G, cg, units); break;
            case 128: walk_phased<128>(r, t, M, (int)G, cg, units); break;
            case 256: walk_phased<256>(r, t, M, (int)G, cg, units); break;
            case 512: walk_phased<512>(r, t, M, (int)G, cg, units); break;
            default: return 2;
          }
        }
      }
    }
    printf("%lld %lld %d\n", (long long)r.lo, (long long)r.hi, lanes);
  }
  return 0;
}
