// Choice of the tiles of a projection launch (host code without HIP).
//
// A launch runs one of three pairs of tiles (modes): large ones for the first
// rows of c and small ones for the rest (gemm.hip).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace kvc {

constexpr int kGemmSlice = 64;     // of K, per slice of a tile's loop
constexpr int kGemmThreads = 512;  // of a workgroup: one tile
constexpr long long kGemmCus = 256;

template <typename T>
constexpr T gemm_div_up(T a, T b) { return (a + b - 1) / b; }

// Measured time of a tile with all CUs busy, in ns: per slice, and once per
// tile.  The latter is the first loads (about 1.5 us) and the store of the
// tile, which every CU does at once where K is short (128 KB, 96 KB, 32 KB or
// 8 KB per CU), less what other workgroups' slices hide where K is long: the
// large tile's is 6.9 us at 4,096 x 16,384 x 128, 7.5 at 8,192 x 8,192 x 1,024
// and 3.9 at 16,200 x 1,024 x 4,096.  The large tiles' values are those that
// choose best: with 8,000 and 7,000, right for stores of 32 bytes a row, 101
// shapes of short K on which the choice differs took 5 % more (754 x 25,640 x
// 576 37 -> 29 us, 1,281 x 4,096 x 512 16.6 -> 14.8), with 5,000 and 4,500 0.5 %.
// Of the 1,500 ns that small tiles once had: narrow outputs of many rows and
// short K took small tiles where large ones are better (42,705 x 256 x 1,024
// 38.7 -> 32.1 us, 42,705 x 256 x 4,096 131 -> 109).  On 440 random shapes (1
// to 23,000 rows, n from 64 to 37,000, k from 64 to 18,800) the launch takes
// 0.43 of the time of 256 x 256 tiles alone with one barrier per slice
// (geometric mean), and at most 3 % more (7,619 x 7,432 x 256).
struct GemmTile {
  int rows, cols;
  long long slice_ns, once_ns;
  constexpr long long time(long long k) const { return slice_ns * (k / kGemmSlice) + once_ns; }
};
// large and small tiles of each mode
constexpr GemmTile kGemmBig[3] = {{256, 256, 1400, 6000}, {256, 192, 1100, 5500}, {128, 128, 480, 4000}};
constexpr GemmTile kGemmSmall[3] = {{128, 128, 480, 4000}, {128, 128, 480, 4000}, {64, 64, 230, 2500}};

// Time until all tiles are done: `big` tiles of cost cb in rounds over the
// CUs, then `small` tiles of cost cs taken by whichever CU is free; cb_cs =
// cb / cs.  (A narrow output of many rows has some 770 splits to try, and a
// division of 64-bit numbers costs ten times the rest of a step.)
inline long long gemm_makespan(long long big, long long cb, long long small, long long cs, long long cb_cs) {
  const long long rounds = big / kGemmCus, extra = big % kGemmCus;  // extra CUs have one large tile more
  const long long early = rounds * cb, late = early + (extra ? cb : 0);
  if (small == 0) return late;
  const long long free_cus = kGemmCus - extra;
  // the CUs that are free early take j small tiles each before the others are free
  const long long j = extra ? cb_cs : 0;
  if (small <= free_cus * j) return std::max(late, early + (long long)gemm_div_up((uint32_t)small, (uint32_t)free_cus) * cs);
  // after that everyone takes tiles; the early ones are at early + j cs <= late
  const long long left = small - free_cus * j, r = left / kGemmCus, rest = left % kGemmCus;
  const long long base_early = early + j * cs;
  long long t = std::max(r > 0 ? (extra ? late : early) + r * cs : late, base_early + r * cs);
  if (rest > 0) t = std::max(t, rest <= free_cus ? base_early + (r + 1) * cs : late + (r + 1) * cs);
  return t;
}

struct GemmPlan {
  int mode;
  long long big_rows;  // row tiles of the larger size
};

// The best split of one mode's tiles, if it takes less than best_t.
template <int MODE>
inline void gemm_best_split(long long m, long long n, long long k, GemmPlan& best, long long& best_t) {
  constexpr GemmTile B = kGemmBig[MODE], S = kGemmSmall[MODE];
  const long long all = gemm_div_up<long long>(m, B.rows), cols = gemm_div_up<long long>(n, B.cols);
  const long long scols = gemm_div_up<long long>(n, S.cols);
  const long long cb = B.time(k), cs = S.time(k), cb_cs = cb / cs;
  const long long window = gemm_div_up(kGemmCus, cols) + 1;
  for (long long r = all; r >= 0 && r >= all - window; --r) {
    const long long rest = r == all ? 0 : m - r * B.rows;
    const long long big = r * cols, small = gemm_div_up<long long>(rest, S.rows) * scols;
    if (big + small > (long long)UINT32_MAX / kGemmThreads) continue;
    const long long t = gemm_makespan(big, cb, small, cs, cb_cs);
    if (best_t < 0 || t < best_t) {
      best_t = t;
      best = {MODE, r};
    }
  }
}

// The tiles, and the split of the rows into large and small ones, with the
// shortest estimated time.  Only the last rows are worth small tiles: as many
// as one round of large ones covers.  It takes the host up to 4 us for outputs
// of at most 256 columns (5.5, 8 to 10 on another CPU, with the tiles' sizes
// as variables and every division in 64 bits), below 0.7 from 1,024 columns on.
inline GemmPlan gemm_plan(long long m, long long n, long long k) {
  GemmPlan best = {0, gemm_div_up(m, 256ll)};
  long long best_t = -1;
  gemm_best_split<0>(m, n, k, best, best_t);
  gemm_best_split<1>(m, n, k, best, best_t);
  gemm_best_split<2>(m, n, k, best, best_t);
  return best;
}

}  // namespace kvc
