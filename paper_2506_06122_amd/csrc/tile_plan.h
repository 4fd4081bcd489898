// The tile kernel's shapes and the choice among them.  Plain integers and floats, used by the launches and - without a
// GPU - by the test that a model's plans are evaluated once.
#pragma once
#include <algorithm>
#include <cmath>

#include "tile_grid.h"

// The tile kernel's shapes.  per_kt, per_kt_alone: microseconds per k-tile of one workgroup's share
// of a CU that holds its full number of workgroups (per_cu), or only one; fixed: what a workgroup
// costs besides (first loads' latency, result), not hidden by a next round when it has the CU to
// itself; start: the launch.  Fitted to 6500 timed launches (17 to 6000 rows, twelve (N, K) pairs of
// the 1.5B, 7B and 30B-A3B shapes, one to sixteen splits; rms error of the log 0.08-0.13); the plans it picks are 1.5 %
// slower than the best of all shapes and splits, where the nine shapes before lost 9 % with the best picks.
struct TileShape {
  int wm, wn, mt, nt, kg, s, per_cu;
  float per_kt, per_kt_alone, start, fixed;
  const char* name[4];  // by epilogue: F32, SWIGLU, LSE, SWIGLU with gathered rows
};
#define TILE_NAME(a) \
  {"gemm_tile_kernel<" a ",0,false>", "gemm_tile_kernel<" a ",1,false>", "gemm_tile_kernel<" a ",3,false>", "gemm_tile_kernel<" a ",1,true>"}
// x-macro: index, template arguments, workgroups per CU, model.  (192 x 256 keeps 192 accumulators a lane and spills some ten
// registers, in its epilogue only.)
#define TILE_SHAPES(X) \
  X(0, 1, 4, 2, 1, 1, 8, 2, 0.113f, 0.123f, 0.82f, 1.15f) /* 32 x 64 */       \
  X(1, 1, 4, 2, 2, 1, 6, 2, 0.185f, 0.191f, 0.91f, 1.49f) /* 32 x 128 */      \
  X(2, 1, 4, 2, 3, 1, 5, 2, 0.257f, 0.259f, 1.78f, 1.51f) /* 32 x 192 */      \
  X(3, 2, 2, 2, 2, 1, 6, 2, 0.165f, 0.165f, 1.76f, 1.16f) /* 64 x 64 */       \
  X(4, 2, 2, 2, 3, 1, 5, 2, 0.212f, 0.217f, 1.47f, 1.55f) /* 64 x 96 */       \
  X(5, 2, 2, 2, 4, 1, 5, 2, 0.243f, 0.239f, 1.65f, 2.06f) /* 64 x 128 */      \
  X(6, 2, 2, 2, 5, 1, 4, 2, 0.285f, 0.288f, 1.72f, 2.27f) /* 64 x 160 */      \
  X(7, 2, 2, 2, 6, 1, 4, 2, 0.315f, 0.315f, 1.92f, 2.60f) /* 64 x 192 */      \
  X(8, 2, 2, 2, 8, 1, 3, 2, 0.381f, 0.475f, 1.05f, 3.95f) /* 64 x 256 */      \
  X(9, 2, 2, 3, 4, 1, 4, 2, 0.304f, 0.306f, 1.76f, 2.70f) /* 96 x 128 */      \
  X(10, 2, 2, 3, 6, 2, 3, 1, 0.383f, 0.383f, 0.13f, 6.99f) /* 96 x 192 */     \
  X(11, 4, 2, 2, 4, 1, 6, 1, 0.382f, 0.382f, 0.00f, 5.61f) /* 128 x 128 */    \
  X(12, 4, 2, 2, 5, 1, 5, 1, 0.440f, 0.440f, 0.00f, 6.44f) /* 128 x 160 */    \
  X(13, 4, 2, 2, 8, 1, 5, 1, 0.587f, 0.587f, 0.00f, 9.17f) /* 128 x 256 */    \
  X(14, 4, 2, 2, 10, 1, 4, 1, 0.714f, 0.714f, 0.00f, 10.21f) /* 128 x 320 */  \
  X(15, 4, 2, 3, 8, 1, 3, 1, 0.833f, 0.833f, 0.00f, 11.44f) /* 192 x 256 */
constexpr TileShape kTileShapes[] = {
#define X(id, wm, wn, mt, nt, kg, s, per_cu, a, b, c, d) \
  {wm, wn, mt, nt, kg, s, per_cu, a, b, c, d, TILE_NAME(#wm "," #wn "," #mt "," #nt "," #kg "," #s)},
    TILE_SHAPES(X)
#undef X
};
constexpr bool grouped_shape(int id) { return id <= 2 || id == 7 || id == 8; }  // the experts' launches (gemm_plan_grouped)
constexpr int kLseMinTile = 8;  // column tiles per workgroup an EPI_LSE launch has at least (sizes the parts' buffers)

// Microseconds one projection is expected to take: the busiest CU's rounds of workgroups, and what comes from beyond the
// L2s - the weights once, the activations once per XCD that works on them (a K split's and row group's share goes to
// one XCD in gcd(splits x row groups, 8) of 8: with 7 or 10 splits every L2 fetches what it would share with 8) -
// joined by their third powers, since neither hides the other entirely; plus reading the split planes back (the next
// launch's work).
inline double tile_cost(const TileShape& t, int M, int n_tiles, int k_tiles, int z) {
  TileGrid g{(int)tile_ceil(n_tiles, t.wn * t.nt), (int)tile_ceil(M, t.wm * t.mt * 16), z};
  const int n = tile_groups(g);
  const int kt = (int)tile_ceil(k_tiles, z), per_cu = t.per_cu, rest = n % per_cu;
  double us = t.start + (double)(n - rest) * (kt * t.per_kt + t.fixed);
  if (rest)
    us += kt * (t.per_kt_alone + (per_cu * t.per_kt - t.per_kt_alone) * (rest - 1) / std::max(1, per_cu - 1)) + t.fixed;
  int sharing = 1;
  while (sharing < 8 && (z * g.gy) % (2 * sharing) == 0) sharing *= 2;
  const double mem = 2.5 + (double)n_tiles * k_tiles * 1024 / 6.0e6 + (double)M * k_tiles * 128 * (8 / sharing) / 5.0e6;
  return std::cbrt(us * us * us + mem * mem * mem) + (double)M * n_tiles * 64 * z / 6.0e6;
}

// What is asked of a plan: M x N x K, at most max_splits K splits, at least min_tiles column tiles to a workgroup.
struct TileAsk {
  int M, N, K, max_splits, min_tiles;
  bool operator==(const TileAsk& o) const {
    return M == o.M && N == o.N && K == o.K && max_splits == o.max_splits && min_tiles == o.min_tiles;
  }
};
struct TileChoice {
  int shape, splits;
};
// tile shape and number of K splits with the lowest expected cost
inline TileChoice tile_choose(const TileAsk& q) {
  const int n_tiles = q.N >> 4, k_tiles = q.K >> 5;
  TileChoice pick{};
  double best = 1e29;
  for (int c = 0; c < (int)(sizeof(kTileShapes) / sizeof(kTileShapes[0])); ++c) {
    const TileShape& t = kTileShapes[c];
    if (t.wn * t.nt < q.min_tiles) continue;
    constexpr int zs[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16};
    for (int z : zs) {
      if (z > 1 && (z > q.max_splits || z * 6 > k_tiles)) break;
      const double us = tile_cost(t, q.M, n_tiles, k_tiles, z);
      if (us < best) {
        best = us;
        pick = TileChoice{c, z};
      }
    }
  }
  return pick;
}
// The choices made last.  Decode steps ask for the same few plans layer after layer, and one takes some 5 us of host time
// (a step of 28 layers and 33 rows 0.6 ms in all, a third of the step).  N and K of a model are multiples of 32 and
// more, so the hash multiplies before it takes the top bits; four ways to a set hold what a model asks for
// at one M (half a dozen plans) even where some of them meet, and of several M the latest.
class TilePlans {
 public:
  long long evaluated = 0;  // calls of tile_choose
  TileChoice operator()(const TileAsk& q) {
    unsigned long long h = 0;
    for (int v : {q.M, q.N, q.K, q.max_splits, q.min_tiles}) h = (h ^ (unsigned)v) * 0x9e3779b97f4a7c15ull, h ^= h >> 29;
    Entry* const set = sets_[(h * 0x9e3779b97f4a7c15ull) >> 58];
    int w = 0;
    while (w < kWays - 1 && !(set[w].ask == q)) ++w;
    Entry e = set[w];  // a hit, or the entry that was asked for longest ago
    if (!(e.ask == q)) {
      e = Entry{q, tile_choose(q)};
      ++evaluated;
    }
    for (; w > 0; --w) set[w] = set[w - 1];
    set[0] = e;
    return e.choice;
  }

 private:
  static constexpr int kWays = 4;
  struct Entry {
    TileAsk ask{};  // M = 0: empty
    TileChoice choice{};
  };
  Entry sets_[64][kWays];
};
