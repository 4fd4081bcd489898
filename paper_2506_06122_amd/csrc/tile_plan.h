// The tile kernel's shapes and the choice among them.  Plain integers and floats, used by the launches and - without a
// GPU - by the test that a model's plans are evaluated once.
#pragma once
#include <algorithm>
#include <cmath>

#include "tile_grid.h"

// The tile kernel's shapes.  per_kt, per_kt_alone: microseconds per k-tile of one workgroup's share
// of a CU that holds its full number of workgroups (per_cu), or only one; fixed: what a workgroup
// costs besides (first loads' latency, result), not hidden by a next round when it has the CU to
// itself; start: the launch; power: microseconds that a k-tile of one workgroup takes of the chip when all CUs are
// busy for long and the power limit sets the clock - 256 x power is 1.15 to 1.4 x per_kt.  The first eleven shapes' times are fitted
// to 6500 launches (17 to 6000 rows, twelve (N, K) pairs of the 1.5B, 7B and 30B-A3B shapes, one to sixteen splits), those of the wide
// wavefronts and every power to 1700 (187 to 10568 rows, eight pairs of the 1.5B and 7B shapes); rms error of the log 0.05-0.13.
// From 187 rows on its picks are 0.8 % behind the best of all shapes measured; the sixteen shapes before, with the power left out, 2.2 %.
// 128 x 128 in eight wavefronts, between 64 x 256 and 96 x 256, saves a round or half a tile where neither fits: 200 x 16384 x 3072
// 49.7 -> 44.8 us, 128 x 27648 x 5120 90.2 -> 81.8, 1000 x 2048 x 5632 in two splits 45.8 -> 40.8.  Of 2744 projections of 13 model
// shapes, 17 to 3600 rows, the picks are 1.1 % behind the best of all shapes.
struct TileShape {
  int wm, wn, mt, nt, kg, s, per_cu;
  float per_kt, per_kt_alone, start, fixed, power;
  const char* name[4];  // by epilogue: F32, SWIGLU, LSE, SWIGLU with gathered rows
};
#define TILE_NAME(a) \
  {"gemm_tile_kernel<" a ",0,false>", "gemm_tile_kernel<" a ",1,false>", "gemm_tile_kernel<" a ",3,false>", "gemm_tile_kernel<" a ",1,true>"}
// Four wavefronts whose ring of stages fills more than half of the LDS: each has a SIMD and its 512 registers to itself.
constexpr bool wide_wavefronts(int wm, int wn, int mt, int nt, int kg, int s) {
  return wm * wn * kg == 4 && 2 * s * kg * (2 * wm * mt + wn * nt) > 160;
}
// x-macro: index, template arguments, workgroups per CU, model.
#define TILE_SHAPES(X) \
  X(0, 1, 4, 2, 1, 1, 8, 2, 0.113f, 0.123f, 0.82f, 1.15f, 0.00019f) /* 32 x 64 */       \
  X(1, 1, 4, 2, 2, 1, 6, 2, 0.185f, 0.191f, 0.91f, 1.49f, 0.00038f) /* 32 x 128 */      \
  X(2, 1, 4, 2, 3, 1, 5, 2, 0.257f, 0.259f, 1.78f, 1.51f, 0.00057f) /* 32 x 192 */      \
  X(3, 2, 2, 2, 2, 1, 6, 2, 0.165f, 0.165f, 1.76f, 1.16f, 0.00038f) /* 64 x 64 */       \
  X(4, 2, 2, 2, 3, 1, 5, 2, 0.212f, 0.217f, 1.47f, 1.55f, 0.00057f) /* 64 x 96 */       \
  X(5, 2, 2, 2, 4, 1, 5, 2, 0.243f, 0.239f, 1.65f, 2.06f, 0.00076f) /* 64 x 128 */      \
  X(6, 2, 2, 2, 5, 1, 4, 2, 0.285f, 0.288f, 1.72f, 2.27f, 0.00096f) /* 64 x 160 */      \
  X(7, 2, 2, 2, 6, 1, 4, 2, 0.315f, 0.315f, 1.92f, 2.60f, 0.00114f) /* 64 x 192 */      \
  X(8, 2, 2, 2, 8, 1, 3, 2, 0.381f, 0.475f, 1.05f, 3.95f, 0.00149f) /* 64 x 256 */      \
  X(9, 2, 2, 3, 4, 1, 4, 2, 0.304f, 0.306f, 1.76f, 2.70f, 0.00115f) /* 96 x 128 */      \
  X(10, 2, 2, 3, 6, 2, 3, 1, 0.383f, 0.383f, 0.13f, 6.99f, 0.00176f) /* 96 x 192 */     \
  X(11, 4, 2, 2, 5, 1, 5, 1, 0.440f, 0.440f, 0.00f, 6.44f, 0.00209f) /* 128 x 160 */    \
  X(12, 2, 2, 3, 8, 1, 5, 1, 0.428f, 0.428f, 1.36f, 5.82f, 0.00219f) /* 96 x 256 */     \
  X(13, 2, 2, 4, 8, 1, 5, 1, 0.541f, 0.541f, 0.69f, 6.99f, 0.00281f) /* 128 x 256 */    \
  X(14, 2, 2, 4, 10, 1, 4, 1, 0.669f, 0.669f, 0.40f, 8.14f, 0.00329f) /* 128 x 320 */   \
  X(15, 2, 2, 5, 8, 1, 4, 1, 0.670f, 0.670f, 0.00f, 8.29f, 0.00336f) /* 160 x 256 */    \
  X(16, 2, 2, 6, 6, 1, 4, 1, 0.610f, 0.610f, 0.00f, 8.00f, 0.00313f) /* 192 x 192 */    \
  X(17, 2, 2, 6, 8, 1, 3, 1, 0.777f, 0.777f, 0.00f, 9.65f, 0.00388f) /* 192 x 256 */       \
  X(18, 4, 2, 2, 4, 1, 6, 1, 0.382f, 0.382f, 0.00f, 5.61f, 0.00167f) /* 128 x 128 */
constexpr TileShape kTileShapes[] = {
#define X(id, wm, wn, mt, nt, kg, s, per_cu, a, b, c, d, e) \
  {wm, wn, mt, nt, kg, s, per_cu, a, b, c, d, e, TILE_NAME(#wm "," #wn "," #mt "," #nt "," #kg "," #s)},
    TILE_SHAPES(X)
#undef X
};
constexpr bool grouped_shape(int id) { return id <= 2 || id == 7 || id == 8; }  // the experts' launches (gemm_plan_grouped)
constexpr int kLseMinTile = 8;  // column tiles per workgroup an EPI_LSE launch has at least (sizes the parts' buffers)

// Microseconds one projection is expected to take: the busiest CU's rounds of workgroups, and what comes from beyond the
// L2s - the weights once, the activations once per XCD that works on them (a K split's and row group's share goes to
// one XCD in gcd(splits x row groups, 8) of 8: with 7 or 10 splits every L2 fetches what it would share with 8) -
// joined by their third powers, since neither hides the other entirely, and no less than the power limit allows (the sixth
// powers: it hardly shows before it binds); plus reading the split planes back (the next launch's work).
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
  const double power = (double)g.nx * g.ny * z * (kt + 8) * t.power;  // a result costs as much as eight k-tiles
  const double both = us * us * us + mem * mem * mem, cube = power * power * power;
  return std::cbrt(std::sqrt(both * both + cube * cube)) + (double)M * n_tiles * 64 * z / 6.0e6;
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
