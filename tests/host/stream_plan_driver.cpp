// CPU-only check of csrc/stream_plan.h: what it picks against measured launches, and the limits of the joined splits.
// Built and run by tests/test_host_tile_grid.py.
#include <cstdio>
#include <vector>

#include "../../paper_2506_06122_amd/csrc/stream_plan.h"

struct Timed {
  int shape, splits;
  double us;
};
// us a launch on an MI355X, weights from HBM; shapes that take more than 1.6 times the best are left out
struct Measured {
  int M, N, K;
  bool joined;
  int max_splits;
  std::vector<Timed> times;
};
static const Measured measured[] = {
    {8, 3072, 1536, false, 1, {{2, 1, 4.9}, {0, 1, 5.2}}},
    {16, 6144, 1536, false, 1, {{2, 1, 9.4}, {0, 1, 6.5}}},
    {16, 12288, 3072, false, 1, {{2, 1, 21.6}, {0, 1, 17.5}}},
    {8, 10240, 512, false, 1, {{0, 1, 4.9}}},
    {17, 3072, 1536, false, 1, {{7, 1, 7.4}, {5, 1, 6.6}}},
    {32, 8192, 2048, false, 1, {{5, 1, 9.7}}},
    {32, 12288, 512, false, 1, {{5, 1, 6.3}}},
    {8, 2048, 1536, false, 4, {{2, 1, 5.3}, {0, 1, 5.1}, {3, 2, 4.2}, {3, 3, 4.1}, {3, 4, 3.8}}},
    {16, 6144, 4096, false, 4, {{2, 1, 17.6}, {0, 1, 12.4}, {3, 2, 14.0}, {3, 3, 14.7}, {3, 4, 13.4}}},
    {1, 6144, 2048, false, 4, {{2, 1, 9.7}, {0, 1, 6.7}, {3, 2, 8.0}, {3, 3, 8.9}, {3, 4, 8.7}}},
    {16, 4608, 4096, false, 4, {{2, 1, 16.9}, {0, 1, 11.8}, {3, 2, 13.2}, {3, 3, 10.8}, {3, 4, 12.2}}},
    {32, 3072, 2048, false, 4, {{7, 1, 8.9}, {5, 1, 8.4}, {8, 2, 6.4}, {8, 3, 8.3}, {8, 4, 7.5}}},
    {32, 6144, 2048, false, 4, {{5, 1, 9.1}, {8, 2, 10.5}, {8, 3, 11.9}, {8, 4, 10.8}}},
    {16, 128, 2048, false, 4, {{2, 1, 5.5}, {3, 2, 4.4}, {3, 3, 3.9}, {3, 4, 3.8}}},
    {8, 1536, 8960, true, 5, {{2, 1, 12.8}, {3, 2, 11.9}, {3, 3, 10.0}, {3, 4, 9.1}, {3, 5, 8.7}, {4, 4, 12.4}}},
    {16, 1536, 1536, true, 5, {{2, 1, 5.2}, {3, 2, 5.6}, {3, 3, 5.7}, {3, 4, 5.3}, {3, 5, 5.6}, {4, 2, 7.6}, {4, 3, 7.2}, {4, 4, 7.1}}},
    {32, 1536, 8960, true, 5, {{7, 1, 15.6}, {8, 3, 13.8}, {8, 4, 11.8}, {8, 5, 11.0}}},
    {8, 4096, 4096, true, 5, {{2, 1, 8.4}, {3, 2, 9.6}, {3, 3, 11.3}, {3, 4, 10.8}, {3, 5, 12.1}, {4, 2, 12.1}, {4, 3, 10.6}, {4, 4, 11.8}}},
    {16, 4096, 12288, true, 5, {{2, 1, 24.2}, {3, 2, 20.8}, {3, 3, 25.6}, {3, 4, 22.1}, {3, 5, 25.5}, {4, 2, 27.9}, {4, 3, 22.8}, {4, 4, 21.7}}},
    {1, 4096, 12288, true, 5, {{2, 1, 19.5}, {3, 2, 19.2}, {3, 3, 22.8}, {3, 4, 20.4}, {3, 5, 22.8}, {4, 2, 25.1}, {4, 3, 21.5}, {4, 4, 21.1}}},
    {8, 3584, 18944, true, 5, {{2, 1, 27.0}, {3, 2, 25.0}, {3, 3, 30.6}, {3, 4, 26.3}, {3, 5, 30.0}, {4, 2, 34.6}, {4, 3, 27.8}, {4, 4, 25.8}}},
    {16, 3584, 18944, true, 5, {{2, 1, 34.6}, {3, 2, 28.3}, {3, 3, 35.0}, {3, 4, 29.8}, {3, 5, 33.8}, {4, 2, 39.2}, {4, 3, 30.5}, {4, 4, 27.1}}},
    {8, 8192, 4096, true, 5, {{2, 1, 15.3}, {3, 2, 16.0}, {3, 3, 17.1}, {3, 4, 18.2}, {3, 5, 19.1}, {4, 2, 18.1}, {4, 3, 19.4}, {4, 4, 20.4}}},
    {16, 5120, 8960, true, 5, {{3, 2, 26.2}, {3, 3, 21.3}, {3, 4, 23.7}, {3, 5, 25.0}, {4, 2, 22.6}, {4, 3, 19.6}, {4, 4, 26.2}}},
    {32, 2048, 2048, true, 5, {{7, 1, 6.0}, {8, 2, 7.2}, {8, 3, 6.7}, {8, 4, 6.3}, {8, 5, 8.5}}},
    {17, 2048, 5632, true, 5, {{7, 1, 9.3}, {8, 2, 11.6}, {8, 3, 10.0}, {8, 4, 9.0}, {8, 5, 11.5}}},
    {8, 512, 2048, true, 5, {{2, 1, 5.0}, {3, 2, 5.6}, {3, 3, 5.3}, {3, 4, 5.2}, {3, 5, 5.3}, {4, 2, 7.7}, {4, 3, 7.1}, {4, 4, 7.0}}},
    {16, 65536, 2048, false, 1, {{0, 1, 45.0}, {1, 1, 52.9}}},
    {8, 65536, 1536, false, 1, {{0, 1, 31.1}, {1, 1, 31.8}}},
    {16, 65536, 1536, false, 1, {{0, 1, 35.5}, {1, 1, 32.1}}},
    {32, 65536, 2048, false, 1, {{5, 1, 58.1}, {6, 1, 48.9}}},
};

int main() {
  int bad = 0;
  for (const Measured& a : measured) {
    const StreamChoice pick = stream_choose(a.M, a.N, a.K, a.joined, a.max_splits);
    double best = 1e9, took = 1e9;
    for (const Timed& t : a.times) {
      if (t.us < best) best = t.us;
      if (t.shape == pick.shape && t.splits == pick.splits) took = t.us;
    }
    if (took > 1.06 * best + 0.1) {  // 0.1 us: the launches' spread
      std::fprintf(stderr, "%d x %d x %d%s: shape %d in %d splits, %.1f us; the best takes %.1f\n", a.M, a.N, a.K, a.joined ? " joined" : "",
                   pick.shape, pick.splits, took, best);
      ++bad;
    }
  }
  int plans = 0;
  for (int joined = 0; joined < 2; ++joined)
    for (int M = 1; M <= 32; ++M)
      for (int N = 32; N <= (joined ? 8192 : 20000); N += 32)
        for (int K = 32; K <= 32768; K += K < 1024 ? 32 : 992)
          for (int most : {1, 3, 16}) {
            const StreamChoice c = stream_choose(M, N, K, joined, most);
            const StreamShape& t = kStreamShapes[c.shape];
            const int blocks = ((N >> 4) + t.nt - 1) / t.nt * ((M + 16 * t.mt - 1) / (16 * t.mt));
            ++plans;
            const bool fine = c.splits >= 1 && c.splits <= (joined ? 5 : most) && (c.splits == 1 || (K >> 5) / c.splits >= 8) &&
                              (!joined || c.splits == 1 || (blocks * t.mt <= kJoinTiles && c.splits * t.nt <= kJoinParts)) &&
                              (M <= 16 || t.mt == 2 || t.keep);
            if (!fine && ++bad < 20) std::fprintf(stderr, "%d x %d x %d joined %d: shape %d, %d splits\n", M, N, K, joined, c.shape, c.splits);
          }
  std::printf("%d plans\n", plans);
  return bad != 0;
}
