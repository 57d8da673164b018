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

// Workgroup id -> tile of a dense launch.  Workgroup ids go round the 8 XCDs one by one, and each XCD takes a run of the tile sequence (they
// differ by one tile at most), in which columns of 8 tile rows follow one another: its 32 workgroups share 8 panels of A and 4 of B.  Grids of a
// number of tiles that 8 does not divide used to go to the XCDs tile by tile, so that every L2 read every panel; us, before -> with this map and what the
// kernel no longer spends ahead of its first load: bf16 321 x 1164 x 8064 (19 x 37 tiles) 24.3 -> 19.5, 393 x 7991 x 1432 23.0 -> 20.1, fp16 310 x 2432 x
// 1408 10.0 -> 7.7; grids that 8 divides gain 0.3 - 0.6 us (1 x 896 x 1664 fp8 3.9 -> 3.4, 512 x 1792 x 1792 fp16 9.05 -> 8.6): two divisions, three fetches of
// arguments one after the other and, at the end, a third of the instructions per stored fragment.
struct TileAt {
  int32_t tm, tn;
};
#if defined(__HIPCC__)
__host__ __device__
#endif
inline TileAt family_tile(uint32_t bid, int32_t grid_m, int32_t grid_n, uint32_t div_group, uint32_t div_last) {
  const uint32_t nwg = (uint32_t)grid_m * (uint32_t)grid_n, q = nwg >> 3, r = nwg & 7, xcd = bid & 7;
  const uint32_t lin = xcd * q + (xcd < r ? xcd : r) + (bid >> 3), per_group = grid_n < 1 << 28 ? 8u * (uint32_t)grid_n : ~0u;
  auto over = [](uint32_t n, uint32_t d, uint32_t f) -> uint32_t { return f ? (uint32_t)(((uint64_t)(2 * n) * f) >> 32) : n / d; };
  const uint32_t group = over(lin, per_group, div_group), in_group = lin - group * per_group, left = (uint32_t)grid_m - 8 * group;
  TileAt t;
  if (left >= 8) {
    t.tm = (int32_t)(8 * group + (in_group & 7)), t.tn = (int32_t)(in_group >> 3);
  } else {
    const uint32_t c = over(in_group, left, div_last);
    t.tm = (int32_t)(8 * group + in_group - c * left), t.tn = (int32_t)c;
  }
  return t;
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
