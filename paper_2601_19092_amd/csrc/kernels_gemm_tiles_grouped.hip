// Grouped GEMM on the 128 x 128 tile of gemm_tiles.h: fp8 groups with fp32 scales, which the matrix cores' scale path cannot
// carry and the grouped tile kernel of that path does not take.  One workgroup per compute unit walks its tiles as one
// pipeline (the loads run on into the next tile's first stages).
//
// What it does not read again: the groups' weights, once tiles replace the streaming kernel's passes of 64 rows over them.  At 1024 tokens of an MoE layer of
// 128 experts (8 per token, N, K = 1536, 2048 gated and 2048, 768) it takes 94 + 56 us for 604 MB of weights (4.3 TB/s): the stream of weights, 0.6 us of a
// K-step's 0.9, beside 0.5 of LDS reads, matrix work and fold, which overlap in part; a ring of five stages is level.  us, first version (a table of 10 us per launch, loads in loops
// over lanes, weights through the caches) -> now: 256 tokens 143 -> 109, 512 tokens 154 -> 119, 1024 tokens 184 -> 148, 4096 tokens 329 -> 297; streaming kernel 1024 tokens 284 + 128.
// Other tiles then, 1024 / 4096 tokens: one tile at a time
// without running on 112 + 85 / 201 + 172; 64 x 128 in four waves, two workgroups per compute unit 105 + 70 / 217 + 151, in eight waves
// 127 + 83 / 278 + 177; 32 x 128 122 + 76 / 290 + 195; 128 x 128 with two stages 163 + 103 / 305 + 198.
#include "gemm_tiles.h"

#include <algorithm>

namespace axe {

namespace {
constexpr TileShape kShape = kTileFamily[kGroupedMember];
template <int GRP, bool ONCE>
void launch(const GemmArgs& g, unsigned nwg, hipStream_t s) {
  hipLaunchKernelGGL((tiles::gemm_tiles_kernel<2, 1, kShape.tm, kShape.tn, kShape.wm, kShape.wn, kShape.wk, kShape.nst, GRP, ONCE>), dim3(nwg),
                     dim3(64 * kShape.wm * kShape.wn * kShape.wk), 0, s, g);
}
}  // namespace

hipError_t launch_gemm_tiles_grouped(const GemmArgs& g0, hipStream_t s) {
  GemmArgs g = g0;
  if (!grouped_tiles_fit(g.N, g.K) || !g.fp8 || !g.scale_a || g.scale_e8m0) return hipErrorInvalidValue;
  g.grid_n = (int32_t)(g.N / kShape.tn);
  const int64_t worst = (g.M / kShape.tm + g.groups) * (int64_t)g.grid_n;
  int64_t nwg = std::max<int64_t>(cu_count(), (worst + 63) / 64);  // a wave keeps the workgroup's tiles one per lane
  nwg = (std::min(nwg, worst) + 7) / 8 * 8;                        // the tile sequence is cut into 8 parts, one per XCD
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  // Weights past the caches where most groups should have one row block: the host's guess from the average, since a second body in this kernel
  // spills.  us: 256 / 512 / 1024 tokens 130 -> 127 / 130 -> 122 / 158 -> 151; guessed wrong, all rows in one group 46.6 -> 47.4, in four 44.7 -> 46.1.
  const bool once = g.stream_b && 2 * g.M <= kShape.tm * (int64_t)g.groups;
  if (g.gated) once ? launch<2, true>(g, (unsigned)nwg, s) : launch<2, false>(g, (unsigned)nwg, s);
  else once ? launch<1, true>(g, (unsigned)nwg, s) : launch<1, false>(g, (unsigned)nwg, s);
  return hipGetLastError();
}

}  // namespace axe
