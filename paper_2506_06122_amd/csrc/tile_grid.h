// How the workgroups of a tile launch cover its blocks.  Plain integers, used by the kernel, by its
// planner and - without a GPU - by the test that every block is visited exactly once.
#pragma once

struct TileGrid {
  int nx = 0, ny = 0, nz = 0;        // column blocks, row blocks, K splits
  int group_m = 1, group_n = 1;      // row and column blocks an XCD takes side by side
  int gy = 1;                        // row groups
  unsigned by_per = 0, by_nz = 0, by_gy = 0, by_m = 0;  // tile_by of group_m * group_n, nz, gy and group_m (tile_divisors)
};
struct TileBlock {
  int x, y, z;
  bool inside;  // false: padding of the XCD-aware launch
};

constexpr long long tile_ceil(long long a, long long b) { return (a + b - 1) / b; }

// x / d for any x and d >= 1, as one multiplication by m = floor(2^32 / d) (2^32 - 1 for d = 1), whose high word is the
// quotient or one less: m is at most 1 below 2^32 / d, so x m / 2^32 is at most x / 2^32 < 1 below x / d.  (A division of
// two runtime integers is some 30 instructions, and the kernel needs four quotients before its first load: 0.3 us of
// a launch.)
constexpr unsigned tile_by(long long d) { return d == 1 ? 0xffffffffu : (unsigned)((1ll << 32) / d); }
constexpr unsigned tile_div(unsigned x, unsigned d, unsigned by) {
  const unsigned q = (unsigned)(((unsigned long long)x * by) >> 32);
  return q + (x - q * d >= d);
}

// Workgroup -> block.  The launch is one-dimensional and workgroups go to the 8 XCDs (each with its own L2)
// round-robin by index, so index % 8 is the XCD and index / 8 the order inside it.  An XCD takes groups of
// group_m row blocks x group_n column blocks, whose workgroups run side by side and share the operands' lines in
// its L2; groups go round the XCDs with the split varying fastest, then the row blocks.
constexpr TileBlock tile_block(const TileGrid& g, unsigned index) {
  const unsigned xcd = index & 7, idx = index >> 3, per = g.group_m * g.group_n, nz = g.nz, gy = g.gy, gm = g.group_m;
  const unsigned run = tile_div(idx, per, g.by_per), unit = run * 8 + xcd, in = idx - run * per;
  const unsigned q = tile_div(unit, nz, g.by_nz), xg = tile_div(q, gy, g.by_gy), xi = tile_div(in, gm, g.by_m);
  const int x = (int)(xg * g.group_n + xi), y = (int)((q - xg * gy) * gm + in - xi * gm);
  return TileBlock{x, y, (int)(unit - q * nz), y < g.ny && x < g.nx};
}
constexpr long long tile_units(const TileGrid& g) { return tile_ceil(g.ny, g.group_m) * tile_ceil(g.nx, g.group_n) * g.nz; }
constexpr long long tile_workgroups(const TileGrid& g) { return tile_ceil(tile_units(g), 8) * 8 * g.group_m * g.group_n; }

// what tile_block divides by, once the launch's groups are set (the planner's search does without)
constexpr void tile_divisors(TileGrid& g) {
  g.by_per = tile_by(g.group_m * g.group_n);
  g.by_nz = tile_by(g.nz);
  g.by_gy = tile_by(g.gy);
  g.by_m = tile_by(g.group_m);
}

// Sets group_m and group_n and returns the workgroups the busiest CU gets (32 CUs to an XCD).
// Groups go to the XCDs whole, so a group that is large against the launch leaves XCDs idle: of the
// group heights that cut the row blocks evenly, the largest with the fewest workgroups per CU.
// With many workgroups in all, four column blocks side by side, so that the group's activation and weight lines
// are both few.
constexpr int tile_groups(TileGrid& g) {
  const int chunks = (int)tile_ceil(g.ny, 16);
  g.group_n = (long long)g.ny * g.nx >= 1024 && g.ny > 4 ? 4 : 1;
  int best = 0x7fffffff, best_m = 1;
  for (int c = chunks; c < chunks + 6 && c <= g.ny; ++c) {
    g.group_m = (int)tile_ceil(g.ny, c);
    const int n = (int)tile_ceil(tile_workgroups(g) / 8, 32);
    if (n < best) {
      best = n;
      best_m = g.group_m;
    }
  }
  g.group_m = best_m;
  g.gy = (int)tile_ceil(g.ny, best_m);
  return best;
}

// The same for the experts' launches.  An expert's few row blocks follow each other (its weights are fetched once),
// and the blocks past the last used one, up to half of them, exit at once.  A row group goes from column to column
// through the XCDs in steps of the number of groups; with 8 groups it meets one XCD in every column, and the unused
// ones left three XCDs idle (14 rows of the 30B-A3B shape: 2.06 ms a step, 12 layers; 1.34 with 9 groups).  So few
// groups come in an odd number (6 -> 7: 1.33 -> 1.27 ms), up to 16 of them not in fours (12 -> 13: 3.23 -> 3.04), and
// more, of which every XCD gets several anyway, not in eights (24 -> 25: 12.7 -> 11.9 ms); cutting 10, 20 or 36
// groups differently as well cost 1 to 3 %.
constexpr bool groups_share_xcds(long long groups) {
  return groups > 1 && groups % (groups < 8 ? 2 : groups < 16 ? 4 : 8) == 0;
}
constexpr void tile_groups_experts(TileGrid& g) {
  const int most = g.ny < 16 ? g.ny : 16;
  g.group_n = 1;
  g.group_m = most;
  while (2 * g.group_m >= most && groups_share_xcds(tile_ceil(g.ny, g.group_m))) --g.group_m;
  if (2 * g.group_m < most) g.group_m = most;
  g.gy = (int)tile_ceil(g.ny, g.group_m);
}
