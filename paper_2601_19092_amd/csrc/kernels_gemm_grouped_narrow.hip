// Grouped GEMM for few rows per group on narrow tiles (gemm_tiles.h): 16, 32 or 64 rows of a group times 64 rows of its B image, all of
// K, two workgroups per compute unit, each walking its tiles as one pipeline.  Any of the library's inputs with plain weights; blocked
// weights, short K, many groups and, in 16 bits, launches of few tiles stay with the streaming kernel (narrow_fits).
//
// What bounds it: HBM, reading the active groups' weights once.  A bare stream of loads into LDS carries 6.75 - 7.0 TB/s through panels of 64 rows
// x 128 bytes with the non-temporal policy (6.2 - 6.3 without, 6.1 - 6.5 through panels of 256 and 128 rows of 4096 bytes), where loads into
// registers in the operand layout -- the streaming kernel -- ask for half lines and lose 10 % with that policy.  Hence weights through
// LDS, whole 128-byte lines, 64 of them per K-step, and rings of 60 - 80 KiB in two workgroups: one's table, first loads and stores lie
// behind the other's stream.
//
// Measured, us, streaming kernel -> this (an MoE layer of 128 experts, 8 per token, both products): fp16 4 / 16 / 64 tokens 51 -> 49 / 125 -> 118 /
// 192 -> 174 (1.15 GB: 6.6 TB/s), 128 tokens 205 -> 183; fp8 (either scales) 1 / 16 / 64 / 128 tokens 17 -> 14 / 73 -> 61 / 108 -> 89 / 128 -> 96.
//
// Weights past the caches where the host says that they don't stay there (stream_b) and the table that most groups have one row block: the second row block
// of a group would read them from memory again.  Two bodies, for a choice at every load costs scaled fp8 7 - 10 % at 8 - 64 tokens.  us, past the caches
// whatever the table says / by the table / through the caches, 128 x 1536 x 2048 (groups x N x K), fp16: 512 rows in sizes drawn around the average 119 / 119 / 134,
// half of them in one group 116 / 115 / 128, in 16 groups 28.3 / 26.2 / 26.2, in four 17.6 / 12.6 / 12.4; 1536 rows in 16 groups 48.4 / 42.2 / 42.1, in one 36.4 / 26.8 / 26.5;
// fp8 512 rows drawn 57.9 / 58.0 / 67.1, in 16 groups 16.8 / 14.4 / 14.3, 1536 rows in four 20.9 / 17.2 / 17.0.
#define AXE_TILES_BODY
#include "gemm_tiles.h"

#include <algorithm>

namespace axe {

namespace tiles {
template <int DT, int SC, int TM, int TN, int WM, int WN, int NST, int GRP>
__global__ __launch_bounds__(64 * WM * WN) void gemm_narrow_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds_mem[NST * (TM + TN) * maps::kLargeRowBytes];
  int t_row0, t_desc;
  if (g.clear && blockIdx.x == 0 && threadIdx.x == 0) *g.clear = 0;
  group_tiles<TM>(g, threadIdx.x & 63, t_row0, t_desc);
  gemm_tiles_body<DT, SC, TM, TN, WM, WN, 1, NST, GRP>(g, (lds_u8)lds_mem, t_row0, t_desc);
}
template <int DT, int SC, int TM, int TN, int WM, int WN, int NST, int GRP>
__global__ __launch_bounds__(64 * WM * WN) void gemm_narrow_by_table_kernel(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds_mem[NST * (TM + TN) * maps::kLargeRowBytes];
  int t_row0, t_desc;
  if (g.clear && blockIdx.x == 0 && threadIdx.x == 0) *g.clear = 0;
  if (group_tiles<TM>(g, threadIdx.x & 63, t_row0, t_desc))
    gemm_tiles_body<DT, SC, TM, TN, WM, WN, 1, NST, GRP, true>(g, (lds_u8)lds_mem, t_row0, t_desc);
  else
    gemm_tiles_body<DT, SC, TM, TN, WM, WN, 1, NST, GRP>(g, (lds_u8)lds_mem, t_row0, t_desc);
}
}  // namespace tiles

namespace {
struct NarrowTile {
  int tm, tn, wm, wn, nst;
};
constexpr NarrowTile kNarrow[] = {{16, 64, 1, 2, kNarrowStages}, {32, 64, 2, 2, kNarrowStages}, {64, 64, 2, 2, kNarrowStages - 1}};

template <int DT, int SC, int V, int GRP>
void launch_as(const GemmArgs& g, unsigned nwg, hipStream_t s) {
  constexpr NarrowTile t = kNarrow[V];
  static_assert(2 * t.nst * (t.tm + t.tn) * maps::kLargeRowBytes <= 160 * 1024, "two workgroups per compute unit");
  const dim3 block(64 * t.wm * t.wn);
  if (g.stream_b) hipLaunchKernelGGL((tiles::gemm_narrow_by_table_kernel<DT, SC, t.tm, t.tn, t.wm, t.wn, t.nst, GRP>), dim3(nwg), block, 0, s, g);
  else hipLaunchKernelGGL((tiles::gemm_narrow_kernel<DT, SC, t.tm, t.tn, t.wm, t.wn, t.nst, GRP>), dim3(nwg), block, 0, s, g);
}

template <int V>
hipError_t launch(const GemmArgs& g0, hipStream_t s) {
  constexpr NarrowTile t = kNarrow[V];
  GemmArgs g = g0;
  g.grid_n = (int32_t)(g.N / t.tn);
  const int64_t worst = (g.M / t.tm + std::min<int64_t>(g.M, g.groups)) * (int64_t)g.grid_n;
  int64_t nwg = std::max<int64_t>(2 * cu_count(), (worst + 63) / 64);   // a wave keeps the workgroup's tiles one per lane
  nwg = (std::min(nwg, worst) + 7) / 8 * 8;                        // the tile sequence is cut into 8 parts, one per XCD
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  const unsigned n = (unsigned)nwg;
  auto go = [&](auto dt, auto sc) {
    if (g.gated) launch_as<decltype(dt)::value, decltype(sc)::value, V, 2>(g, n, s);
    else launch_as<decltype(dt)::value, decltype(sc)::value, V, 1>(g, n, s);
  };
  using std::integral_constant;
  if (!g.fp8 && g.f16) go(integral_constant<int, 1>{}, integral_constant<int, 0>{});
  else if (!g.fp8) go(integral_constant<int, 0>{}, integral_constant<int, 0>{});
  else if (!g.scale_a) go(integral_constant<int, 2>{}, integral_constant<int, 0>{});
  else if (!g.scale_e8m0) go(integral_constant<int, 2>{}, integral_constant<int, 1>{});
  else go(integral_constant<int, 2>{}, integral_constant<int, 3>{});
  return hipGetLastError();
}
}  // namespace

hipError_t launch_gemm_grouped_narrow(const GemmArgs& g, hipStream_t s) {
  if (!narrow_fits(g)) return hipErrorInvalidValue;
  const int rows = narrow_rows(g);
  return rows == 16 ? launch<0>(g, s) : (rows == 32 ? launch<1>(g, s) : launch<2>(g, s));
}

}  // namespace axe
