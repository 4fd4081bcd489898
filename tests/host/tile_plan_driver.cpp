// CPU-only check of csrc/tile_plan.h: a forward pass asks for the same few plans layer after layer, and each is
// evaluated once.  Built and run by tests/test_host_tile_grid.py.
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

int main() {
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
