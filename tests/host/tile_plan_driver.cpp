// CPU-only check of csrc/tile_plan.h: a forward pass asks for the same few plans layer after layer, and each is
// evaluated once; tiles of 128 x 128 are picked where they measured best.  Built and run by tests/test_host_tile_grid.py.
#include <cstdio>
#include <vector>

#include "../../paper_2506_06122_amd/csrc/tile_plan.h"

struct Model {
  const char* name;
  int layers, hidden, q_dim, kv_dim, ffn, experts, vocab;
};

// the projections of a step of M rows in launch order, as the forward pass asks for them
static std::vector<TileAsk> step(const Model& m, int M) {
  std::vector<TileAsk> asks;
  for (int l = 0; l < m.layers; ++l) {
    asks.push_back({M, m.q_dim + 2 * m.kv_dim, m.hidden, 16, 0});
    asks.push_back({M, m.hidden, m.q_dim, 16, 0});
    if (m.experts) {
      asks.push_back({M, m.experts, m.hidden, 16, 0});
    } else {
      asks.push_back({M, 2 * m.ffn, m.hidden, 1, 0});
      asks.push_back({M, m.hidden, m.ffn, 16, 0});
    }
  }
  asks.push_back({M, m.vocab, m.hidden, 1, 0});
  return asks;
}

// projections whose fastest tile is 128 x 128 by 8 to 12 % (us on an MI355X, it / the best of the others)
struct Fastest {
  int M, N, K, max_splits;
  double us, others;
};
static const Fastest square[] = {{200, 16384, 3072, 1, 44.8, 49.7},  {256, 16384, 3072, 1, 46.6, 51.0}, {128, 27648, 5120, 1, 81.8, 90.2},
                                 {1000, 2048, 5632, 2, 40.8, 45.8}, {1200, 3072, 512, 1, 10.4, 11.7},  {2100, 1536, 1536, 1, 22.0, 24.8}};

int main() {
  for (const Fastest& f : square) {
    const TileShape& t = kTileShapes[tile_choose(TileAsk{f.M, f.N, f.K, f.max_splits, 0}).shape];
    if (t.wm * t.mt != 8 || t.wn * t.nt != 8) {
      std::fprintf(stderr, "%d x %d x %d: a tile of %d x %d, not the one of 128 x 128\n", f.M, f.N, f.K, t.wm * t.mt * 16, t.wn * t.nt * 16);
      return 1;
    }
  }
  const Model models[] = {{"1.5B", 28, 1536, 1536, 256, 8960, 0, 151936},
                          {"7B", 28, 3584, 3584, 512, 18944, 0, 152064},
                          {"30B-A3B", 48, 2048, 4096, 512, 0, 128, 151936},
                          {"small", 24, 512, 512, 256, 1536, 0, 8192}};
  for (const Model& m : models) {
    const long long kinds = m.experts ? 4 : 5;
    TilePlans plans;
    long long want = 0;
    for (int M = 17; M < 700; M = M < 300 ? M + 1 : M + 7) {
      for (int again = 0; again < 2; ++again)  // the next step has as many rows, or a few samples fewer
        for (const TileAsk& q : step(m, M)) {
          const TileChoice got = plans(q), ref = tile_choose(q);
          if (got.shape != ref.shape || got.splits != ref.splits) {
            std::fprintf(stderr, "%s: %d x %d x %d: shape %d in %d splits, not %d in %d\n", m.name, q.M, q.N, q.K, got.shape, got.splits, ref.shape, ref.splits);
            return 1;
          }
        }
      want += kinds;
      if (plans.evaluated != want) {
        std::fprintf(stderr, "%s, %d rows: %lld plans evaluated so far, not %lld\n", m.name, M, plans.evaluated, want);
        return 1;
      }
    }
    std::printf("%s: %lld plans\n", m.name, plans.evaluated);
  }
  return 0;
}
