// The streamed projections' shapes and the choice between them: plain integers and floats, used by the launcher and -
// without a GPU - by its test.
#pragma once
#include <algorithm>

// Column tiles (16 outputs) per workgroup nt, row tiles mt, k-tiles in flight ku, wavefronts nw; keep: the weights stay in the L2s.
// What a launch is expected to take, in us: start, then for every round of 256 workgroups (one to a CU) `round` and kt for each k-tile
// of a workgroup, and `all` for each k-tile of 1000 workgroups (what they have from memory in common).  kt and all: up to 8 rows, whose
// fragments are half as many lines, and more.  Fitted to 6366 launches, weights from HBM: 128 to 12288 outputs, K 512 to 18944, 1 to 32
// rows, one to five splits; rms error of the log 0.034.  Its picks are 0.2 % behind the best of the shapes
// measured, 18 % at worst; one rule by the bytes of a CU, fitted to six launches, was 2 % behind, and 41 % where its splits filled
// the CUs with small pieces (4096 x 4096, 4 rows: 11.8 us instead of 8.4).
struct StreamShape {
  int mt, nt, ku, nw;
  bool keep;
  float start, round, kt[2], all[2];
  const char* name[3];  // by epilogue: F32, SWIGLU, RESID
};
// x-macro: index, template arguments, the epilogues each is planned with, model (none for the shapes that a rule picks)
#define STREAM_SHAPES(X)                                                                                                             \
  X(0, 1, 2, 2, 8, false, EPI_F32, EPI_SWIGLU_BF16, 2.428f, 0.202f, 0.0453f, 0.0592f, 0.108f, 0.099f) /* outputs in one piece */      \
  X(1, 1, 4, 1, 8, false, EPI_F32, EPI_F32, 0, 0, 0, 0, 0, 0)                                         /* the logits from 9 rows on */  \
  X(2, 1, 1, 3, 16, false, EPI_F32, EPI_RESID, 1.293f, 1.695f, 0.0297f, 0.0426f, 0.048f, 0.046f)      /* narrow, in one piece */      \
  X(3, 1, 2, 3, 8, false, EPI_F32, EPI_RESID, 1.956f, 0.915f, 0.0422f, 0.0545f, 0.133f, 0.129f)       /* K splits: planes, or joined */ \
  X(4, 1, 4, 2, 8, false, EPI_RESID, EPI_RESID, 1.159f, 2.760f, 0.0732f, 0.0912f, 0.269f, 0.240f)     /* K splits, joined */          \
  X(5, 2, 2, 2, 4, false, EPI_F32, EPI_SWIGLU_BF16, 2.511f, 0.321f, 0.0713f, 0.0713f, 0.120f, 0.120f) /* 17 to 32 rows, in one piece */ \
  X(6, 2, 4, 1, 4, false, EPI_F32, EPI_F32, 0, 0, 0, 0, 0, 0)                                         /* the logits */               \
  X(7, 1, 1, 3, 16, true, EPI_F32, EPI_RESID, 1.558f, 1.446f, 0.0312f, 0.0312f, 0.041f, 0.041f)       /* narrow, a row block per 16 rows */ \
  X(8, 2, 2, 2, 8, false, EPI_F32, EPI_RESID, 1.863f, 1.194f, 0.0732f, 0.0732f, 0.128f, 0.128f)       /* K splits */
#define STREAM_NAME(a) {"gemm_stream_kernel<" a ",0>", "gemm_stream_kernel<" a ",1>", "gemm_stream_kernel<" a ",2>"}
constexpr StreamShape kStreamShapes[] = {
#define X(id, mt, nt, ku, nw, keep, e0, e1, start, round, kt8, kt16, all8, all16) \
  {mt, nt, ku, nw, keep, start, round, {kt8, kt16}, {all8, all16}, STREAM_NAME(#mt "," #nt "," #ku "," #nw "," #keep)},
    STREAM_SHAPES(X)
#undef X
};

// joined: the splits meet in the launch, 0.9 us and 0.17 for each (as planes, which the next launch sums, they cost next to nothing)
inline double stream_cost(const StreamShape& t, int M, int N, int K, int splits, bool joined) {
  auto up = [](int a, int b) { return (a + b - 1) / b; };
  const int kt = up(K >> 5, splits), z = up(K >> 5, kt), wgs = up(N >> 4, t.nt) * up(M, 16 * t.mt) * z, more = M > 8;
  return t.start + up(wgs, 256) * (t.round + t.kt[more] * kt) + t.all[more] * 1e-3 * wgs * kt + (joined && z > 1 ? 0.908 + 0.17 * z : 0.0);
}

// Scratch of the K splits that meet in their launch (join_splits): at most kJoinTiles joined tiles, each of at most
// kJoinParts KiB, and as many tickets.
constexpr int kJoinTiles = 512, kJoinParts = 16;

struct StreamChoice {
  int shape, splits;
};
// Shape and number of K splits with the lowest expected cost; joined: the projection adds to the residual.  Each split has
// at least 8 k-tiles; four column tiles not where K is a multiple of 4096: the tiles are 128 KiB and more apart then and share memory
// channels (8192 x 4096, 8 rows: 18.1 us in two splits, 14.3 expected, 16.0 with two column tiles, 15.4 in one piece).
//
// The logits of 16384 ids and more are workgroups enough in one piece: two column tiles to a workgroup, four as soon as the
// activations weigh as much as the weights, but up to 16 rows not where the tiles are a multiple of 64 KiB apart (memory channels again).
// 65536 outputs, us with two / four:  K 1536: 8 rows 31.1 / 31.8, 16 rows 35.5 / 32.1, 32 rows 48.1 / 37.6;
//                                     K 2048: 8 rows 40.3 / 49.9, 16 rows 45.0 / 52.9, 32 rows 58.1 / 48.9.
inline StreamChoice stream_choose(int M, int N, int K, bool joined, int max_splits) {
  if (!joined && N >= 16 * 1024) return StreamChoice{M > 16 ? 6 : M > 8 && K % 2048 ? 1 : 0, 1};
  struct Range {
    int shape, least, most;  // splits
  };
  static constexpr Range ranges[2][2][3] = {{{{2, 1, 1}, {0, 1, 1}, {3, 2, 4}}, {{7, 1, 1}, {5, 1, 1}, {8, 2, 4}}},
                                            {{{2, 1, 1}, {3, 2, 5}, {4, 2, 4}}, {{7, 1, 1}, {8, 2, 5}, {8, 1, 0}}}};
  StreamChoice pick{};
  double best = 1e29;
  for (const Range& r : ranges[joined][M > 16]) {
    if (r.shape == 4 && K % 4096 == 0) continue;
    for (int z = r.least; z <= std::min(r.most, joined ? r.most : max_splits) && (z == 1 || (K >> 5) / z >= 8); ++z) {
      const double us = stream_cost(kStreamShapes[r.shape], M, N, K, z, joined);
      if (us < best) {
        best = us;
        pick = StreamChoice{r.shape, z};
      }
    }
  }
  return pick;
}
