// Which tile takes a call, from its sizes alone. Plain host code: the launches are in qgemm_api.hip and
// moe_direct.hip, and the CPU tests compile this file by itself.
#pragma once

#include <algorithm>

namespace qg {

enum class DenseTile { k256x256, k256x128, k128x256, k128x128 };

struct DensePlan {
  DenseTile tile;
  int splits;      // workgroups that share a tile's K
};

constexpr int kMinStepsPerSplit = 12;

inline long ceil_div(long a, long b) { return (a + b - 1) / b; }

// Whether a launch can have so many workgroups. The runtime counts a grid's threads in 32 bits and does not
// refuse more: a launch of 2^24 + 1484 workgroups of 256 threads returned success and ran 1484 of them.
inline bool grid_fits(long workgroups, int threads) { return workgroups <= 0xffffffffL / threads; }

// Splits of nk K steps, at most `most` (and eight), each of at least kMinStepsPerSplit steps.
inline int k_splits(long most, long nk) {
  int S = (int)std::max<long>(1, std::min<long>(8, most));
  while (S > 1 && nk / S < kMinStepsPerSplit) --S;
  return S;
}

// The dense GEMM above the small-M kernel.
//
// 256x256 tiles from 200 of them on. Up to 1024 rows with fewer: eight-wave tiles of half that size, twice
// the tiles, so half the K split and half the fp32 partials; the split keeps tiles x splits <= 256 (one
// workgroup per CU, one round). Up to 2048 rows only where one of the two forms has more than 128 tiles.
// Fewer 256x256 tiles but a long K: K split over several workgroups per tile so that every CU gets one.
//
// Below 256 rows the half-size tile is 128x256. From there on 256x128 dequantises each weight for twice the
// rows, but the two cover the same output with different numbers of tiles, so one of them may need a second
// round of workgroups or afford fewer splits of K. The cost is counted in K steps of a 256x128 workgroup:
// rounds x steps, a 128x256 step 1.3 (Q4) or 1.5 (Q8) of them, and for a split the second launch (6) and its
// partials (1 per 2^20). Over 320 calls of 256 to 2048 rows in both formats the pick is at most 6% slower
// than 128x256 throughout and, but for one call (11%), at most 2.5% slower than 256x128 throughout; it is 10%
// and 9% faster on average. Measured, 128x256 against 256x128 (us, * the one taken):
//   as many rounds and steps   Q4 512x8192x3072 42.2, 39.6*  1536x4096x4096 69.2, 62.6*  768x1536x2048 25.5, 22.7*
//                              Q8 512x2048x2048 24.2, 23.5*  2048x4096x2048 44.9, 41.6*
//   one round against two      Q4 1100x7168x2048 41.7*, 58.2  640x11008x4096 69.4*, 99.8  1904x4285x3040 62.3*, 93.7
//                              Q8 1100x7168x2048 53.3*, 61.1  1028x6912x2048 40.4*, 55.2  637x11848x6528 174, 171*
//   two splits against one     Q4 576x6340x3360 42.7*, 46.0  590x5760x7200 73.9*, 111  259x8396x1632 27.3, 24.5*
//                              Q8 576x6340x3360 50.9, 49.4*  590x5760x7200 104*, 132  352x8964x1888 33.0, 28.5*
//   three splits against two   Q4 600x4096x4096 36.1*, 36.7  Q8 600x4096x4096 44.5, 38.0*
// and 256x128 against 256x256: Q8 2048x2048x8192 85.6, 82.6* (two splits against four), 2048x8192x2048 80.4,
// 69.0*. Above 1024 rows a 256x128 form with at most 128 tiles takes the call only if it splits K: Q8
// 1506x2688x7616 80.7* against 194 unsplit as 128x256, but Q4 1154x3088x576 13.1 against 12.2* as 128x128.
inline DensePlan dense_plan(bool q4, long M, long N, long K) {
  const long nk = ceil_div(K, 64);
  const long big = ceil_div(M, 256) * ceil_div(N, 256);
  if (M >= 256 && N >= 256 && big >= 200) return {DenseTile::k256x256, 1};
  const bool vec = M * N % 4 == 0;         // the partials are summed four at a time
  if (M >= 128 && M <= 2048 && N >= 256 && vec) {
    const long wide = ceil_div(M, 128) * ceil_div(N, 256);
    const int ws = k_splits(256 / wide, nk);
    if (M < 256) return {DenseTile::k128x256, ws};
    const long tall = ceil_div(M, 256) * ceil_div(N, 128);
    const int ts = k_splits(256 / tall, nk);
    auto cost = [&](long tiles, int S, double step) {
      const double sums = S > 1 ? 6 + (double)S * M * N / (1 << 20) : 0;
      return ceil_div(tiles * S, 256) * ceil_div(nk, S) * step + sums;
    };
    if (M <= 1024 || tall > 128 || (wide > 128 && ts > 1)) {
      if (cost(tall, ts, 1.0) <= cost(wide, ws, q4 ? 1.3 : 1.5)) return {DenseTile::k256x128, ts};
      return {DenseTile::k128x256, ws};
    }
  }
  if (M >= 256 && N >= 256 && vec) {
    const int S = k_splits(ceil_div(256, big), nk);
    if (S > 1) return {DenseTile::k256x256, S};
  }
  return {DenseTile::k128x128, 1};
}

// The direct MoE kernel (moe_direct.hpp): one 32-row block of weights per wave, `waves` of them and so
// 32 x waves columns per workgroup (fused gate/up 16 x waves of h).
constexpr int kMoeSlice = 128;   // experts per launch

inline int moe_direct_waves(int rows) { return rows == 64 ? 8 : 4; }

inline long moe_direct_tiles(int rows, bool swi, long cols) {
  return ceil_div(cols, (swi ? 16 : 32) * moe_direct_waves(rows));
}

// Upper bound of sum_e ceil(c_e / rows): every active expert (at most one per row) adds one group and its
// further rows whole groups.
inline long moe_direct_groups(int rows, long M, long experts) {
  const long active = std::min(experts, M);
  return (M - active) / rows + active;
}

// Rows per group of the direct kernel for M rows over E experts and cols output columns, 0 where the staged
// tiles take the call. From the mean rows per expert (the host does not see the routing).
// Taller groups dequantise a large expert's weights fewer times, shorter ones leave more workgroups
// and registers for loads in flight; four waves per workgroup spread few items over more CUs.
// Measured on E=128 top-8 hidden 2048 inter 768 Q4 (gate/up + SiLU, down; us), against the staged
// tiles that took these calls before (64x128 / 128x128 up to 32 rows, 192x256 above):
//   T=4    32-row 19.6, 9.8     64-row 20.8, 10.4    staged 27.5, 17.0
//   T=128  32-row 66.9, 34.2    64-row 67.9, 35.4    128-row 77.5, 42.6   staged 96.0, 57.4
//   T=500  32-row 94.6, 54.7    64-row 86.3, 50.5    128-row 93.7, 59.4   staged 114, 75.4
//   T=1024 64-row 119, 73.5     128-row 114, 77.4    staged 124, 81.6
//   T=1536 64-row 149, 93.2     128-row 135, 96.4    staged 137, 95.1
// and E=64 top-6 hidden 2048 inter 1056 Q8 (its 64-row form spills; 32-row up to a mean of 32):
//   T=300 (mean 28)   32-row 83.8, 51.6   128-row 87.5, 48.5   staged 105, 57.2
//   T=777 (mean 73)   32-row 166, 88.6    128-row 106, 65.4    staged 160, 78.7
//   T=1200 (mean 112) 128-row 127, 90.6   staged 167, 86.1
inline int moe_direct_rows(bool q4, bool swi, long M, long E, long cols) {
  const long mean = M / E;
  if (mean > (q4 ? 80 : 96)) return 0;
  const int rows = mean <= (q4 ? 16 : 32) ? 32 : q4 && mean <= 48 ? 64 : 128;
  // the staged tiles are larger, and so their grids smaller
  const long items = moe_direct_groups(rows, M, std::min<long>(E, kMoeSlice)) * moe_direct_tiles(rows, swi, cols);
  return grid_fits(items, 64 * moe_direct_waves(rows)) ? rows : 0;
}

}  // namespace qg
