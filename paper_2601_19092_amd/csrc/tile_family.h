// The family of small and medium workgroup tiles (gemm_tiles.h): their shapes, and which of them a problem takes.
// Plain host and device code.
#pragma once
#include <stdint.h>

namespace axe {

// tm x tn = the workgroup's tile of C, wm x wn = its wave grid, wk = groups of wm x wn waves that take alternate
// K-tiles (their sums meet in LDS at the end), nst = stages of the ring in LDS (a stage: one K-tile per group).
struct TileShape {
  int tm, tn, wm, wn, wk, nst;
};
constexpr TileShape kTileFamily[] = {
    {16, 16, 1, 1, 8, 4},    // one fragment per wave, K dealt to eight waves: a decode step's few rows against many weights
    {16, 32, 1, 1, 8, 3},
    {32, 16, 1, 1, 8, 3},
    {32, 32, 1, 1, 4, 4},
    {64, 32, 2, 1, 4, 3},
    {64, 64, 2, 2, 2, 4},
    {128, 64, 4, 2, 1, 5},
    {128, 128, 4, 2, 1, 4},
    {256, 128, 4, 2, 1, 3},
};
constexpr int kTileFamilySize = sizeof kTileFamily / sizeof kTileFamily[0];

// Division by a divisor that the host knows, on 32 bits: n / d = (2 n f) >> 32 with f = ceil(2^31 / d), exact for all n <= most where most d < 2^31: f is less
// than 1 above 2^31 / d, so n f / 2^31 is less than n / 2^31 < 1 / d above n / d and reaches no next whole number.  0: out of that range, divide.
inline uint32_t div_factor(uint64_t d, uint64_t most) {
  return d == 0 || most >= (uint64_t(1) << 31) / d ? 0 : (uint32_t)(((uint64_t(1) << 31) + d - 1) / d);
}

// What the map below needs of a grid, worked out by the host.
enum : uint32_t { kRuns = 0, kBlocks = 1, kInTurn = 2 };
struct TileMap {
  uint32_t div_group, div_last;   // div_factor() of the tiles of a group of 8 tile rows, and of the last group's tile rows (kBlocks: of the blocks of a row)
  uint32_t deal;                  // how the tiles go to the XCDs: kRuns, kBlocks (of 16 x 16) or kInTurn (tile by tile)
  uint32_t turns;                 // 4 bits for each XCD: the tile columns by which its run is turned
};
// Where a launch is four rounds of tiles and more, every XCD walks along its rows of C at the pace of the others.  Runs that start at one or two columns (grid_m a
// multiple of 32), or whole multiples of 16 tile columns apart (4 KiB of a row of C in 16 bits), write the same few of the memory's channels at any time; dealt in blocks, the 256 tiles
// of a round are 16 columns side by side.  us, runs / blocks: fp8 8176 x 4096 (32 x 32 tiles) K 512 50.0 / 45.9 with fp32 scales, unscaled K 1024 63.3 / 62.1, 8176 x 8192 K 512
// E8M0 93.3 / 86.2, 4080 x 8192 (16 x 64) 48.2 / 46.4; bf16 8176 x 8188 x 512 129 / 115.  Others start spread out and are faster in runs: 12272 x 4092 x 512 (48 x 32) bf16
// 83.6 / 91.4, 20464 x 4096 x 1024 (80 x 32) fp8 128 / 154, 8176 x 2044 x 2048 (32 x 16, two rounds) bf16 69.4 / 72.6.
//
// Turns, for the same reason, where 8 does not divide the tiles, three rounds and more (to 64: the largest timed has 10): XCD x begins its run 4 x columns past a multiple of 16 (its share of a round is 4
// columns) and ends with what it skipped.  Round robin / runs / turned, us: fp8 31 x 31 tiles 7842 x 3908 x 512 with fp32 scales 40.7 / 44.4 / 42.0, unscaled 7776 x 3968 x 768 52.3 /
// 50.9 / 48.4, bf16 31 x 33 7840 x 4220 x 512 67.7 / 58.8 / 54.3; over 107 products of 18 such grids 1 / 0.934 / 0.925 of the time, the slowest turned 29 x 29 with scales
// (7286 x 3652 x 512 36.7 / 38.2 / 38.0), the slowest run 1.09.  (Where 8 divides them the runs start as they always have.)
//
// One round of tiles that 8 does not divide goes in turn unless the XCDs then read many more rows (rows_read; 15 % decide, since the count leaves out when they are read): an XCD
// has one row of every group of 8 tile rows, all columns of it, so few XCDs read a panel of A, where a run that goes from one group into the next reads up to 16.  us, in turn / runs: bf16 6733 x 244 x 8128
// (53 x 4 tiles of 128 x 64) 41.0 / 52.5, 3284 x 332 x 2088 (26 x 6) 13.2 / 18.0, f16 711 x 475 x 3208 (12 x 15 of 64 x 32) 11.1 / 13.6, 2578 x 67 x 6160 (81 x 3 of 32 x 32) 13.7 / 16.6, 15243 x 64 x 1216 (239 x 1 of
// 64 x 64) 8.4 / 9.2, fp8 2275 x 793 x 2224 (18 x 13 of 128 x 64) 10.4 / 11.7; and bf16 3002 x 51 x 2088 (94 x 2) 7.0 / 6.5.  Of 815 such launches of all members 607 go in turn; 0.3 % slower than the faster way on average, always in runs
// 1.8 %, always in turn 0.8 %.  With more rounds it decides less (three of 92 more than 3 % slower in runs), and a grid of up to 8 tile rows has a single group.
//
// Rows of A and B that the XCDs read between them, each panel once for every XCD that has a tile of it; grid_m > 8.
inline int64_t rows_read(uint32_t deal, int64_t grid_m, int64_t grid_n, int64_t tm, int64_t tn) {
  const int64_t group = 8 * grid_n, tiles = grid_m * grid_n, q = tiles / 8, r = tiles % 8, full = grid_m / 8, last = grid_m % 8;
  int64_t rows = 0, cols = 0;
  for (int64_t x = 0; x < 8; ++x) {
    if (deal == kInTurn) {                                           // of the last group, position x and every 8th from there
      const int64_t has = last ? (last * grid_n - x + 7) / 8 : 0, all = last % 4 == 0 ? 1 : (last % 2 ? last : last / 2);
      rows += full + (has < all ? has : all), cols += grid_n;
      continue;
    }
    int64_t at = x * q + (x < r ? x : r), end = at + q + (x < r), lo = 0, hi = 0, next = 0;   // its first piece has columns lo .. hi, the others 0 .. next - 1
    for (bool first = true; at < end; first = false) {
      const int64_t g = at / group, start = g * group, height = g < full ? 8 : last, stop = end < start + height * grid_n ? end : start + height * grid_n;
      rows += stop - at < height ? stop - at : height;
      const int64_t c = (stop - 1 - start) / height;
      if (first) lo = (at - start) / height, hi = c;
      else next = c + 1 > next ? c + 1 : next;
      at = stop;
    }
    cols += next <= lo ? next + hi - lo + 1 : (next > hi + 1 ? next : hi + 1);
  }
  return rows * tm + cols * tn;
}
inline TileMap family_runs(int64_t grid_m, int64_t grid_n) {
  const uint64_t group = 8 * (uint64_t)grid_n;
  return {div_factor(group, (uint64_t)grid_m * (uint64_t)grid_n), div_factor((uint64_t)(grid_m & 7), group), kRuns, 0};
}
inline TileMap family_map(int64_t grid_m, int64_t grid_n, int64_t tm, int64_t tn, int64_t round) {   // tiles of tm x tn, round of them at a time
  const uint64_t tiles = (uint64_t)grid_m * (uint64_t)grid_n, group = 8 * (uint64_t)grid_n, q = tiles / 8, r = tiles % 8;
  TileMap m = family_runs(grid_m, grid_n);
  if (((grid_m | grid_n) & 15) == 0 && tiles >= 1024 && (grid_m % 32 == 0 || tiles % 1024 == 0)) m.deal = kBlocks, m.div_last = div_factor((uint64_t)grid_n / 16, tiles / 256);
  if (r != 0 && grid_m > 8 && tiles <= (uint64_t)round && 20 * rows_read(kInTurn, grid_m, grid_n, tm, tn) < 23 * rows_read(kRuns, grid_m, grid_n, tm, tn)) m.deal = kInTurn;
  for (uint64_t x = 0; x < 8 && r != 0 && grid_m >= 8 && q >= 96 && q <= 2048; ++x) {
    const uint64_t first = x * q + (x < r ? x : r), turn = (4 * x - first % group / 8) & 15;
    if (8 * turn < q) m.turns |= (uint32_t)turn << (4 * x);
  }
  return m;
}

// Workgroup id -> tile of a dense launch.  Workgroup ids go round the 8 XCDs one by one, and each XCD takes a run of the tile sequence (they
// differ by one tile at most; other deals above), in which columns of 8 tile rows follow one another: its 32 workgroups share 8 panels of A and 4 of B.  Grids of a
// number of tiles that 8 does not divide used to go to the XCDs tile by tile, all of them; us, before -> with this map and what the
// kernel no longer spends ahead of its first load: bf16 321 x 1164 x 8064 (6 x 37 tiles) 24.3 -> 19.5, 393 x 7991 x 1432 23.0 -> 20.1, fp16 310 x 2432 x
// 1408 10.0 -> 7.7; grids that 8 divides gain 0.3 - 0.6 us (1 x 896 x 1664 fp8 3.9 -> 3.4, 512 x 1792 x 1792 fp16 9.05 -> 8.6): two divisions, three fetches of
// arguments one after the other and, at the end, a third of the instructions per stored fragment.
struct TileAt {
  int32_t tm, tn;
};
#if defined(__HIPCC__)
__host__ __device__
#endif
inline TileAt family_tile(uint32_t bid, int32_t grid_m, int32_t grid_n, const TileMap& map) {
  const uint32_t xcd = bid & 7, pos = bid >> 3;
  auto over = [](uint32_t n, uint32_t d, uint32_t f) -> uint32_t { return f ? (uint32_t)(((uint64_t)(2 * n) * f) >> 32) : n / d; };
  TileAt t;
  if (map.deal == kBlocks) {
    const uint32_t per_row = (uint32_t)grid_n >> 4, block = pos >> 5, row = over(block, per_row, map.div_last), at = block - row * per_row;
    t.tm = (int32_t)(16 * row + 8 * (xcd >> 2) + (pos & 7)), t.tn = (int32_t)(16 * (row & 1 ? per_row - 1 - at : at) + 4 * (xcd & 3) + (pos >> 3 & 3));
    return t;
  }
  const uint32_t nwg = (uint32_t)grid_m * (uint32_t)grid_n, q = nwg >> 3, r = nwg & 7, run = q + (xcd < r ? 1 : 0);
  const uint32_t turned = pos + 8 * (map.turns >> (4 * xcd) & 15), in_run = xcd * q + (xcd < r ? xcd : r) + (turned < run ? turned : turned - run);
  const uint32_t lin = map.deal == kInTurn ? bid : in_run;
  const uint32_t per_group = grid_n < 1 << 28 ? 8u * (uint32_t)grid_n : ~0u;
  const uint32_t group = over(lin, per_group, map.div_group), in_group = lin - group * per_group, left = (uint32_t)grid_m - 8 * group;
  if (left >= 8) {
    t.tm = (int32_t)(8 * group + (in_group & 7)), t.tn = (int32_t)(in_group >> 3);
  } else {
    const uint32_t c = over(in_group, left, map.div_last);
    t.tm = (int32_t)(8 * group + in_group - c * left), t.tn = (int32_t)c;
  }
  return t;
}

// Whether a member's reads and loads have places of their own between the matrix instructions (gemm_tiles.h; sc: 0 unscaled, 1 fp32 scales, 2 E8M0 codes).
// The 256 x 128 tile's sixteen fragments a wave: left to the compiler, a stage's reads gather behind its products and the next barrier waits for
// them.  Placed, us: bf16 2048 x 4096 x 2048 36.8 -> 34.9, fp16 to fp32 2299 x 2950 x 4040 72.1 -> 68.5, fp8 2048 x 4096 x 4096 36.5 -> 34.3.  Smaller tiles are level either
// way (128 x 128 at 2000 x 2000 x 2048 18.8 / 18.7, 1024 x 3584 x 8192 57.9 / 58.7), and so is this one with fp32 scales, whose fold stands between the products
// (1000 x 3584 x 8192 63.0 / 66.4).  E8M0 codes have their products added up behind them: unplaced / placed K 512 4080 x 12288 69.2 / 71.6, 2040 x 4096 12.0 / 12.2, K 1024 and 1536
// level, K 2048 4080 x 4092 41.6 / 41.3, K 4096 2000 x 4096 37.7 / 37.1, K 8192 3000 x 5000 128 / 123.
// (Unscaled, two rounds of tiles and 6 to 10 K-tiles: it goes by the card.  bf16 4080 x 4092 x 512 unplaced / placed 25.5 / 24.3 on one, 27.0 / 28.1 on another.)
constexpr bool family_placed(int member, int sc, int64_t K) {
  const TileShape t = kTileFamily[member];
  return t.tm * t.tn >= 256 * 128 && (sc == 0 || (sc == 2 && K >= 2048));
}

// The member that serves grouped problems (one wave group: the pipeline runs on from tile to tile), and the problems it takes:
// whole tiles along N, counted in 11 bits, and at least as many K-tiles of 128 as its ring has stages.
constexpr int kGroupedMember = 7;
static_assert(kTileFamily[kGroupedMember].wk == 1, "no partial sums");
inline bool grouped_tiles_fit(int64_t N, int64_t K) {
  const TileShape& t = kTileFamily[kGroupedMember];
  return N % t.tn == 0 && N / t.tn <= 2048 && K % 128 == 0 && K / 128 >= t.nst;
}

}  // namespace axe
