// How the workgroups of a tile launch cover its blocks.  Plain integers, used by the kernel, by its
// planner and - without a GPU - by the test that every block is visited exactly once.
#pragma once

struct TileGrid {
  int nx = 0, ny = 0, nz = 0;        // column blocks, row blocks, K splits
  int group_m = 1, group_n = 1;      // row and column blocks an XCD takes side by side
};
struct TileBlock {
  int x, y, z;
  bool inside;  // false: padding of the XCD-aware launch
};

constexpr long long tile_ceil(long long a, long long b) { return (a + b - 1) / b; }

// Workgroup -> block.  The launch is one-dimensional and workgroups go to the 8 XCDs (each with its own L2)
// round-robin by index, so index % 8 is the XCD and index / 8 the order inside it.  An XCD takes groups of
// group_m row blocks x group_n column blocks, whose workgroups run side by side and share the operands' lines in
// its L2; groups go round the XCDs with the split varying fastest, then the row blocks.
constexpr TileBlock tile_block(const TileGrid& g, unsigned index) {
  const int xcd = index & 7, idx = index >> 3, per = g.group_m * g.group_n;
  const int unit = (idx / per) * 8 + xcd, in = idx % per;
  const int gy = (g.ny + g.group_m - 1) / g.group_m, q = unit / g.nz;
  const int x = (q / gy) * g.group_n + in / g.group_m, y = (q % gy) * g.group_m + in % g.group_m;
  return TileBlock{x, y, unit % g.nz, y < g.ny && x < g.nx};
}
constexpr long long tile_units(const TileGrid& g) { return tile_ceil(g.ny, g.group_m) * tile_ceil(g.nx, g.group_n) * g.nz; }
constexpr long long tile_workgroups(const TileGrid& g) { return tile_ceil(tile_units(g), 8) * 8 * g.group_m * g.group_n; }

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
  while (g.group_m > most / 2 && groups_share_xcds(tile_ceil(g.ny, g.group_m))) --g.group_m;
  if (g.group_m <= most / 2) g.group_m = most;
}
