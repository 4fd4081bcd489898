// CPU-only check of csrc/tile_grid.h: the workgroups of a tile launch visit every (column block, row block, K split)
// exactly once, for every shape of launch the planner can ask for.  Built and run by tests/test_host_tile_grid.py.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2506_06122_amd/csrc/tile_grid.h"

static void check(const TileGrid& g, const char* what) {
  const long long n = tile_workgroups(g);
  std::vector<unsigned char> seen((size_t)g.nx * g.ny * g.nz, 0);
  for (long long i = 0; i < n; ++i) {
    const TileBlock b = tile_block(g, (unsigned)i);
    if (!b.inside) continue;
    if (b.x < 0 || b.y < 0 || b.z < 0 || b.z >= g.nz || seen[((size_t)b.z * g.ny + b.y) * g.nx + b.x]++) {
      std::fprintf(stderr, "%s %d x %d x %d in groups of %d x %d: workgroup %lld\n", what, g.nx, g.ny, g.nz, g.group_m, g.group_n, i);
      std::exit(1);
    }
  }
  for (unsigned char s : seen)
    if (s != 1) {
      std::fprintf(stderr, "%s %d x %d x %d in groups of %d x %d: a block is missing\n", what, g.nx, g.ny, g.nz, g.group_m, g.group_n);
      std::exit(1);
    }
}

// tile_div against the division, around multiples of the divisor up to the last 32-bit number
static bool quotients() {
  for (long long d : {1ll, 2ll, 3ll, 5ll, 7ll, 12ll, 16ll, 61ll, 64ll, 641ll, 1000ll, 4095ll, 4883ll, 65535ll, 65537ll, 1000003ll, 0x7fffffffll})
    for (long long step : {1ll, 3ll, 1009ll, 65537ll, 1000003ll})
      for (long long k = 0; k < 2000; ++k)
        for (long long at : {k * step * d, 0x80000000ll - k * step * d, 0x100000000ll - k * step * d, 0x100000000ll - k * step})
          for (long long x = at - 2; x <= at + 2; ++x)
            if (x >= 0 && x < 0x100000000ll && tile_div((unsigned)x, (unsigned)d, tile_by(d)) != (unsigned)(x / d)) {
              std::fprintf(stderr, "%lld / %lld\n", x, d);
              return false;
            }
  return true;
}

int main() {
  int n = 0;
  if (!quotients()) return 4;
  // the last workgroups of a launch far larger than any this library makes
  {
    TileGrid g;
    g.nx = 4099, g.ny = 200003, g.nz = 1;
    tile_groups(g);
    tile_divisors(g);
    const long long last = tile_workgroups(g);
    for (long long i = last > 3000000 ? last - 3000000 : 0; i < last; ++i) {
      const long long idx = i >> 3, per = (long long)g.group_m * g.group_n, unit = idx / per * 8 + (i & 7), in = idx % per;
      const long long gy = tile_ceil(g.ny, g.group_m), x = unit / gy * g.group_n + in / g.group_m, y = unit % gy * g.group_m + in % g.group_m;
      const TileBlock b = tile_block(g, (unsigned)i);
      if (b.x != x || b.y != y || b.z != 0) return 5;
    }
  }
  const int wide[] = {1, 2, 3, 5, 8, 12, 13, 28, 36, 112, 140, 148, 297, 594, 1187, 1188};
  for (int nx : wide)
    for (int ny : {1, 2, 3, 4, 5, 6, 7, 15, 16, 17, 31, 33, 64, 100, 129, 289, 513})
      for (int nz : {1, 2, 3, 7, 16}) {
        if ((long long)nx * ny * nz > 700000) continue;
        TileGrid g;
        g.nx = nx, g.ny = ny, g.nz = nz;
        const int per_cu = tile_groups(g);
        tile_divisors(g);
        check(g, "dense");
        // the busiest XCD's workgroups, shared by its 32 CUs
        if ((long long)per_cu * 256 < (long long)nx * ny * nz || g.group_m < 1 || g.group_m > 16) return 2;
        if (nz == 1) {  // the experts' launches
          tile_groups_experts(g);
          tile_divisors(g);
          check(g, "grouped");
        }
        ++n;
      }
  // the used row blocks of an experts' launch come first: whatever their share, no XCD gets much more than an
  // eighth of their workgroups (a third more where 12 columns meet 8 XCDs; with groups of 16 throughout it was up to 3.4 times as much)
  for (int nx : {8, 12, 16})
    for (int ny = 8; ny <= 600; ++ny)
      for (int used : {(2 * ny + 4) / 5, (7 * ny + 9) / 10, ny}) {
        TileGrid g;
        g.nx = nx, g.ny = ny, g.nz = 1;
        tile_groups_experts(g);
        tile_divisors(g);
        int load[8] = {};
        for (long long i = 0; i < tile_workgroups(g); ++i) {
          const TileBlock b = tile_block(g, (unsigned)i);
          load[i & 7] += b.inside && b.y < used;
        }
        for (int l : load)
          if (ny > 20 && l * 8.0 > 1.45 * nx * used) {
            std::fprintf(stderr, "%d of %d row blocks, %d columns: an XCD gets %d workgroups of %d\n", used, ny, nx, l, nx * used);
            return 3;
          }
      }
  std::printf("%d launches\n", n);
  return 0;
}
