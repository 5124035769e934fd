// Which tile takes a call, from its sizes alone. Plain host code: the launches are in qgemm_api.hip and
// moe_direct.hip, and the CPU tests compile this file by itself.
#pragma once

#include <algorithm>

namespace qg {

enum class DenseTile { k256x256, k256x128, k128x256, k128x128 };

struct DensePlan {
  DenseTile tile;
  int splits;      // workgroups that share a tile's K
  int keep;        // splits that the workspace of partials is to hold, at least those
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
  if (M >= 256 && N >= 256 && big >= 200) return {DenseTile::k256x256, 1, 1};
  const bool vec = M * N % 4 == 0;         // the partials are summed four at a time
  if (M >= 128 && M <= 2048 && N >= 256 && vec) {
    const long wide = ceil_div(M, 128) * ceil_div(N, 256);
    const int ws = k_splits(256 / wide, nk);
    if (M < 256) return {DenseTile::k128x256, ws, ws};
    const long tall = ceil_div(M, 256) * ceil_div(N, 128);
    const int ts = k_splits(256 / tall, nk);
    auto cost = [&](long tiles, int S, double step) {
      const double sums = S > 1 ? 6 + (double)S * M * N / (1 << 20) : 0;
      return ceil_div(tiles * S, 256) * ceil_div(nk, S) * step + sums;
    };
    if (M <= 1024 || tall > 128 || (wide > 128 && ts > 1)) {
      // a call on 256x128 tiles also keeps what the splits of the other tiles would take
      const int other = M <= 1024 || wide > 128 ? ws : k_splits(ceil_div(256, big), nk);
      if (cost(tall, ts, 1.0) <= cost(wide, ws, q4 ? 1.3 : 1.5)) return {DenseTile::k256x128, ts, std::max(ts, other)};
      return {DenseTile::k128x256, ws, std::max(ws, other)};
    }
  }
  if (M >= 256 && N >= 256 && vec) {
    const int S = k_splits(ceil_div(256, big), nk);
    if (S > 1) return {DenseTile::k256x256, S, S};
  }
  return {DenseTile::k128x128, 1, 1};
}

struct SmallPlan {
  long splits;     // workgroups along K per 32-row block
  long cps;        // chunks of K per split
  long keep;       // splits that the workspace of partials is to hold, at least those
};

constexpr long kSmTargetGroups = 256;   // workgroups (of eight waves) to fill the CUs without a K split
constexpr int kSmChunks = 8 * 8;        // chunks that a workgroup's eight waves hold in registers at most

// The small-M kernel (qgemm_smallm.hpp) for MT column blocks, P row blocks and K in chunks of kc.
//
// M <= 16 (or up to 128 in MT blocks of 16 columns): 32 weight rows per workgroup; K is split over
// workgroups only when there are fewer than 256 row blocks (or a wave would hold more than eight
// chunks) and K is longer than small_unsplit_k. Split partials go to the split-K workspace and a
// second kernel adds them in split order: a dependent launch (about 2 us) and a partial per output and
// workgroup, so a short K is faster in one workgroup's hands and a long one in few. One block: about
// 1024 of K to a workgroup (two Q8 chunks or one Q4 chunk per wave); two blocks 512; more blocks at
// least 4 chunks, as their matrix work per chunk is larger. Measured in captured graphs, splits filling
// 256 workgroups (with several blocks: of 4 chunks at least) against this rule (us):
//   1 row     Q4 2048x2048 5.7 -> 4.7, 6000x2048 6.6 -> 5.1, 512x8192 8.0 -> 6.4; Q8 1000x512 6.0 -> 2.9,
//             512x2048 7.6 -> 5.0, 300x2560 9.1 -> 5.6, 1500x4128 7.7 -> 6.8
//   16 rows   Q4 1024x1024 6.9 -> 3.8, 7168x2048 8.2 -> 6.4; Q8 4096x2048 7.1 -> 6.6, 768x6144 10.3 -> 7.6
//   24 rows   Q4 1024x1024 6.0 -> 4.6, Q8 2048x512 5.5 -> 3.8, 256x2048 6.7 -> 5.9 (unsplit 7.2)
//   64 rows   Q8 1024x512 6.3 -> 5.1; unsplit at K = 1024 256 columns 7.1 against 6.3, 2048 7.1 against 7.6
//   128 rows  Q8 1024x512 8.3 -> 7.2; unsplit at K = 1024 11.0 against 9.4
constexpr int small_unsplit_k(int MT) { return MT == 1 ? 2048 : MT == 2 ? 1024 : 512; }

inline SmallPlan small_plan(int MT, long P, long K, long kc) {
  const long nc = ceil_div(K, kc);
  const long fill = std::min(nc, ceil_div(kSmTargetGroups, P));
  const long few = MT == 1 ? fill : std::min(fill, std::max<long>(1, nc / 4));   // at least 4 chunks each
  long S = few;
  if (K <= small_unsplit_k(MT)) S = 1;
  else if (MT == 1) S = std::min(S, ceil_div(K, 1024));
  else if (MT == 2) S = std::min({fill, nc / 4, ceil_div(K, 512)});
  auto even = [&](long s) {      // no part empty, none longer than the registers hold
    const long cps = ceil_div(nc, std::max(s, ceil_div(nc, kSmChunks)));
    return SmallPlan{ceil_div(nc, cps), cps, 0};
  };
  SmallPlan p = even(S);
  p.keep = std::max(p.splits, even(few).splits);
  return p;
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
// and registers for loads in flight; four waves per workgroup spread few items over more CUs. So 32 rows
// while the mean is small, and further while the next height would leave the chip idle: Q4, one 64-row
// workgroup (eight waves) per CU, above a mean of 32, where an expert takes two 32-row groups, one per two CUs;
// Q8, three 128-row workgroups per two CUs. Over 200 random calls whose height these limits moved (8 to 128
// experts, 17 to 80 rows on average, random logits with or without a Zipf bias; gate/up and down together)
// the Q4 ones take 0.74 of the time that they take with limits on the mean alone (16, 48; the slowest 1.04),
// the Q8 ones 0.94 (32; 1.07).
// Measured (gate/up + SiLU, down; us) on routing by random logits, against the staged tiles that took these
// calls before (64x128 / 128x128 up to a mean of 32 rows, 192x256 above; * the one taken):
//   Q4 E=128 top-8 2048/768   T=128  32-row 65.2, 29.4*  64-row 60.2, 31.4   128-row 73.6, 38.6   staged 92.9, 54.5
//                             T=512  32-row 85.8, 44.6   64-row 77.3, 42.1*  128-row 88.1, 50.1   staged 99.5, 64.7
//                             T=1024 32-row 133, 82.7    64-row 115, 70.9    128-row 112, 72.3*   staged 122, 79.7
//   Q4 E=256 top-8 4096/2048  T=512  32-row 629, 353     64-row 630, 345*   128-row 737, 397     staged 870, 570
//     the same with a Zipf bias      32-row 389, 221     64-row 345, 194*   128-row 355, 201     staged 456, 259
//   Q4 E=8 top-2 4096/2048    T=128  32-row 35.6, 21.3*  64-row 46.2, 26.9   128-row 39.9, 23.2   staged 42.8, 29.8
//   Q8 E=64 top-6 2048/1056   T=128  32-row 76.1, 39.3*  128-row 79.7, 40.1   staged 99.7, 50.2
//                             T=300  32-row 88.4, 48.8   128-row 87.0, 45.1*  staged 104, 53.9
//                             T=777  32-row 159, 87.4    128-row 104, 60.9*   staged 158, 70.5
// The Q8 64-row form is left out: it spills 41 (gate/up) and 37 (down) of its 128 VGPRs, the 32-row one 4 and
// 5. With most rows on a few experts the mean says too little: all on a quarter or an eighth of the experts at
// means of 40 to 80 the staged tiles, which are then full, are the faster ones, by up to 1.45 times on one
// launch (Q4 E=128 T=640 on 32 experts 64.9, 36.8 against 46.5, 31.0), where routing by random logits gains as
// much (81.3, 51.1 against 113, 72.9) and a Zipf bias over the experts a fifth (78.4, 45.4 against 99.5, 52.6).
// With top-1 a Zipf bias concentrates enough to lose, too (Q4 E=96 2368/1184 T=3746 152 together against 132).
inline int moe_direct_rows(bool q4, bool swi, long M, long E, long cols) {
  const long mean = M / E;
  if (mean > (q4 ? 80 : 96)) return 0;
  // workgroups of the next height if every active expert had the mean
  const int taller = q4 ? 64 : 128;
  const long active = std::min(M, E);
  const long items = active * ceil_div(M / active, taller) * moe_direct_tiles(taller, swi, cols);
  int rows;
  if (q4) {
    const bool low = (mean <= 16 && M < 4096) || items < (mean <= 32 ? 256 : 128);
    rows = low ? 32 : mean <= 48 ? 64 : 128;
  } else {
    const bool low = mean <= 20 || (mean <= 32 && items <= 384);
    rows = low ? 32 : 128;
  }
  // the staged tiles are larger, and so their grids smaller
  const long grid = moe_direct_groups(rows, M, std::min<long>(E, kMoeSlice)) * moe_direct_tiles(rows, swi, cols);
  return grid_fits(grid, 64 * moe_direct_waves(rows)) ? rows : 0;
}

// Prefill attention (attn_kernels.hpp) with few workgroups: whether each owns 64 query rows, not 128, and two
// waves share a query's keys. That halves the chain of key blocks and doubles the workgroups, at more work per
// block. Two workgroups fit a CU (four with D = 64), so it pays
//   - up to one 64-row workgroup per CU; one key block has no chain to halve (S <= 64), and without the mask a
//     second block of a few keys does not pay either;
//   - up to two per CU where that many 128-row ones do not fit one per CU either, or where the chains are long
//     enough; D = 64 up to four. The 64-row form takes the heaviest blocks of all heads first, dealt to the
//     XCDs evenly only for a multiple of 8 heads: others stop earlier;
//   - causal, D = 128: beyond that where the chains are long and uneven.
// Measured, 128-row against 64-row (us, * the one taken; S x heads of all batches, a fourth as many key heads):
//   D=128 causal  64 x 64 5.9*, 6.4  96 x 64 7.9, 6.6*  96 x 320 10.7*, 13.3  192 x 128 9.4*, 9.9  300 x 96 14.5, 11.3*
//                 512 x 32 14.6, 11.7*  512 x 128 22.8*, 25.2  700 x 64 21.1*, 21.6  2048 x 16 39.2, 32.9*
//   D=128 full    65 x 160 7.2*, 8.8  128 x 64 7.8, 7.1*  192 x 128 9.6*, 10.1  512 x 64 16.3, 16.1*  2048 x 32 69.2*, 79.9
//   D=64  causal  96 x 256 6.5, 5.9*  96 x 640 9.1*, 10.5  300 x 192 12.7, 10.3*  1024 x 64 19.3, 18.6*
// Over 1425 calls (32 to 2048 rows, 8 to 640 heads) 4 are more than 3% slower than 128 rows throughout, the worst
// 6%, and the time is 0.939 of it on average; limits on the number of 128-row workgroups alone (causal 400, 640
// with D = 64; full 256), without a look at S, made 217 of them slower, by up to 27%, and came to 0.953.
inline bool attn_split(bool d64, bool causal, long S, long heads) {
  const long wide = heads * ceil_div(S, 128), narrow = heads * ceil_div(S, 64);
  const bool even = heads % 8 == 0;
  if (S <= 64) return false;
  if (!causal) return S > 72 && (S <= 450 ? narrow : wide) <= 256;
  if (narrow <= 256) return true;
  if (d64) return narrow <= (S <= 128 ? 768 : S <= 320 || (!even && S > 600) ? 1024 : even ? 1200 : 600);
  if (wide > 256)
    return narrow <= 528 || (S > 600 && even && wide <= 320) || (S >= 900 && wide <= (S < 1200 ? 384 : 400));
  return (S > 128 && S <= 160) || (S > 192 && (even || S > 600 || narrow <= 400));
}

}  // namespace qg
