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

// The member that serves grouped problems (one wave group: the pipeline runs on from tile to tile), and the problems it takes:
// whole tiles along N, counted in 11 bits, and at least as many K-tiles of 128 as its ring has stages.
constexpr int kGroupedMember = 7;
static_assert(kTileFamily[kGroupedMember].wk == 1, "no partial sums");
inline bool grouped_tiles_fit(int64_t N, int64_t K) {
  const TileShape& t = kTileFamily[kGroupedMember];
  return N % t.tn == 0 && N / t.tn <= 2048 && K % 128 == 0 && K / 128 >= t.nst;
}

}  // namespace axe
