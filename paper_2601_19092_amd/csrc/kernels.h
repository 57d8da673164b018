// Launch entry points of the kernels (host-callable; defined in the .hip files).
#pragma once
#include <hip/hip_runtime.h>
#include <stdlib.h>

#include "device_types.h"

namespace axe {

// HIP refuses a launch of 2^32 threads or more: workgroups of 256 that one launch holds
constexpr uint64_t kMaxBlocks256 = (uint64_t(1) << 24) - 1;

hipError_t launch_layout_eval(const EvalDesc& d, int64_t n, const int64_t* idx, int64_t* out, hipStream_t s);
// Whether an evaluation that the fast kernel does not take goes by blocks of indices.  A thread of the block kernel writes a pair of words
// per trip, a trip whole indices and an even number of words: per <= 256, so more than half of the threads write (an odd per of
// 129 .. 169 leaves two of the three indices that fit; 52 % at 133).  Pairs start on 16 bytes.  More words per index leave few whole
// indices to a trip and long runs to a thread: the general kernel keeps those, and index spaces of 2^31 points and more -- and a
// few indices with such an odd per, whose half trips a handful of workgroups would make one after the other (1536 indices, 43 replicas on 3
// axes: 20.6 us on the general kernel, 25.8 by blocks; 10000: 21.8 and 27.4; 90300: 74 and 35; 1536, 129 replicas on one axis: 46 and 25).
inline bool layout_eval_by_blocks(const EvalDesc& d, int64_t n, const int64_t* out) {
  const int64_t per = d.E_R * d.n_axes;
  const bool half_trips = (per & 1) && 512 / per == 3;
  return d.use32 && per <= 256 && ((uintptr_t)out & 15) == 0 && !(half_trips && n < 16384 && d.E_R <= 64);
}
hipError_t launch_relayout_joint(const RelayoutPlan& p, int unit_bytes, const void* src, void* dst, hipStream_t s);
// elem_bytes 1, 2, 4 or 8; rows of at least 16 bytes; a workgroup takes kRowSlots slots, and one launch holds kMaxBlocks256 workgroups
constexpr uint64_t kRowSlots = 16;
hipError_t launch_relayout_rows(const RowPlan& p, int elem_bytes, const void* src, void* dst, hipStream_t s);
// elem_bytes 1, 2, 4 or 8; every 16-byte chunk of a tile row must be aligned on both sides
hipError_t launch_relayout_transpose(const TransposePlan& p, int elem_bytes, const void* src, void* dst, hipStream_t s);
// tile edge (elements) the transposing kernel uses for an element size
// (measured on 8192 x 8192: rows of 256 - 512 bytes per tile beat 128-byte rows by 10 - 17 %, except for
//  single bytes, where the gather of 16 LDS bytes per store makes a 256 x 256 tile slower)
inline int transpose_tile_edge(int elem_bytes) { return elem_bytes == 8 ? 64 : 128; }
// tile of its skewed variant, elements along the source and along the destination.  Measured, 8191 x 8193 bf16, us: 64 x 128 56, 64 x 256
// 58, 128 x 192 63, 64 x 192 65, 128 x 128 66; 5001 x 7001 fp32: 64 x 128 63, 32 x 192 65, 64 x 192 69, 32 x 128 72, 32 x 96 75.
constexpr int skew_tile_s(int elem_bytes) { return elem_bytes == 8 ? 32 : 64; }
constexpr int skew_tile_d(int elem_bytes) { return elem_bytes == 8 ? 64 : 128; }
hipError_t launch_relayout_generic(const GenericRelayoutPlan& p, int unit_bytes, const void* src, void* dst,
                                   hipStream_t s);
// a member of the tile family (tile_family.h)
hipError_t launch_gemm_tiles_16bit(int member, const GemmArgs& g, hipStream_t s);
// fp8 groups with fp32 scales on the tile family; grouped_tiles_fit(N, K)
hipError_t launch_gemm_tiles_grouped(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_tiles_fp8(int member, const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_small(const GemmArgs& g, bool fp8, hipStream_t s);
// Large-tile kernels: 256 x tile_n workgroup tile (tile_n = 256, or 224 for bf16); require
// M % 256 == 0, N % tile_n == 0 and K a multiple of the K step (bf16: 64, fp8: 128).
hipError_t launch_gemm_bf16_256(const GemmArgs& g, hipStream_t s);
// grouped (g.group_rows, g.groups, g.ldg set; g.M = rows of all groups together, any value): N % 256 == 0, K % 64 == 0
hipError_t launch_gemm_bf16_256_grouped(const GemmArgs& g, hipStream_t s);
// two grouped problems, the second reading the first's output, as one launch with tile-level hand-over (Sec. 4.1,
// fused MoE layer); sync = M + 1 words of device memory.  need_extra (tests only) raises the count a wait expects,
// so that with a small spin_limit every wait gives up.
// rows the library's own pair workspace serves, and its address on the current device (no allocation: a __device__ array)
constexpr int64_t kPairStaticRows = int64_t(1) << 20;
hipError_t pair_static_workspace(int32_t** out);
hipError_t launch_pair_sync_clear(int32_t* p, int64_t n, hipStream_t s);   // p[0 .. n) = 0, by a small kernel
// rows: of a tile, 128, 192 or 256 (pair_tile_rows)
hipError_t launch_gemm_bf16_256_grouped_pair(const GemmArgs& g1, const GemmArgs& g2, int rows, int32_t* sync, int spin_limit, int need_extra,
                                             hipStream_t s);
// dense with ragged edges through the grouped kernel (g.groups = 1, g.group_rows null): any M, N % 8 == 0, K % 64 == 0
hipError_t launch_gemm_bf16_256_ragged(const GemmArgs& g, hipStream_t s);
// rows of a tile of the grouped tile kernel: 128 unless the groups are large on average (the host knows M, not the
// group sizes) or tile_m says otherwise.  Measured on an MoE layer (128 groups, N = 1536, K = 2048 and N = 2048,
// K = 768): 128-row tiles win by 2 - 11 % up to 64 rows per group on average, draw at 256, and lose 3 - 4 % at 512 and
// 7 - 8 % from 1024 on (AXE_GROUPED_TILE128_ROWS overrides the threshold for experiments).
struct Tile128Rows {
  int avg;
  bool set;
};
inline Tile128Rows grouped_tile128_rows() {
  static const Tile128Rows r = [] { const char* v = getenv("AXE_GROUPED_TILE128_ROWS"); return Tile128Rows{v ? atoi(v) : 384, v != nullptr}; }();
  return r;
}
inline int grouped_tile_rows(int64_t M, int groups, int tile_m) {
  if (tile_m) return tile_m == 128 ? 128 : 256;
  return M <= (int64_t)grouped_tile128_rows().avg * groups ? 128 : 256;
}
// The same choice for the fp8 grouped tile kernel (AXE_GROUPED_FP8_TILE128_ROWS overrides the threshold).  Measured on
// the same layer with E8M0 scales (gemm1 + gemm2, us, 256-row against 128-row tiles): 16 rows per group 158 against 136,
// 32 rows 163 against 140, 128 rows 224 against 190, 256 rows 281 against 274, 512 rows 429 against 439, 1024 rows 722
// against 775.
inline int grouped_fp8_tile_rows(int64_t M, int groups, int tile_m) {
  static const int small_avg = [] { const char* v = getenv("AXE_GROUPED_FP8_TILE128_ROWS"); return v ? atoi(v) : 384; }();
  if (tile_m == 128 || tile_m == 256) return tile_m;
  return M <= (int64_t)small_avg * groups ? 128 : 256;
}
// grouped, few rows per group: one workgroup per (group, 128 rows of B), weights streamed once, no LDS
hipError_t launch_gemm_grouped_stream(const GemmArgs& g, hipStream_t s);
// the same on narrow tiles whose weights pass through LDS; narrow_fits(g)
hipError_t launch_gemm_grouped_narrow(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_fp8_256(const GemmArgs& g, hipStream_t s);
// fp8 with E8M0 block scales (or none) on the matrix cores' scale path; same shape requirements
hipError_t launch_gemm_fp8_e8m0_256(const GemmArgs& g, hipStream_t s);
hipError_t launch_gemm_fp8_e8m0_256_grouped(const GemmArgs& g, hipStream_t s);

// Compute units of the current device (host side; asked once per process).
inline int cu_count() {
  static int cus = 0;
  if (!cus) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus = n;
  }
  return cus;
}

// The burst variant of the 64 x 64 kernel serves 16-bit problems made of whole 64 x 64 tiles with at most 8 K-tiles of 64
// (K <= 512), C rows aligned for the vector stores, and few enough tiles that they are all on the chip at once (a workgroup
// holds 16 KiB of LDS per K-tile, so at most one or two fit a compute unit: with many tiles the regular kernel's higher
// occupancy wins).
inline bool small_preload_fits(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
  static const bool enabled = [] { const char* v = getenv("AXE_SMALL_BURST"); return !v || atoi(v) != 0; }();
  if (!enabled || M % 64 || N % 64 || K % 64 || K > 512 || K <= 0) return false;
  if (ldc % 4 || 64 * lda * 2 >= (int64_t(1) << 31) || 64 * ldb * 2 >= (int64_t(1) << 31)) return false;
  return (M / 64) * (N / 64) <= cu_count();
}

// Whether the narrow tiles take a grouped problem of few rows per group from the streaming kernel: plain weights, at least as many K-tiles as their ring
// has stages, tile columns that fit the table's 11 bits; and where they are the faster ones.  us, streaming / narrow, weights out of the caches (and the same
// weights again and again), every group as large as the others or drawn around the average with weights exp(N(0, 1/2)):
//   - the table costs every workgroup a pass over the groups: 4096 x 256 x 1152 (groups x N x K) fp16 4 rows per group 398 / 403, 1 row 243 / 267, fp8
//     135 / 160; 512 x 1024 x 1024 fp16 177 / 162, fp8 96 / 84.
//   - fp8: the streaming kernel splits K by two only.  Scaled, 8 x 1024 x 1024 (128 tiles) 2 rows 7.9 / 5.9 (4.9 / 5.0), 4 x 1024 x 1024 (64) 7.4 / 5.5 (4.9 / 5.0),
//     1 x 256 x 1024 (4) 5.9 / 5.1 (4.8 / 4.9), x 2048 9.7 / 6.7 (7.4 / 6.5), x 4096 17 / 9.9 (12 / 9.8).  With 768 of K the same weights again are 0.3 us faster there:
//     128 x 2048 x 768, 8 of the groups with a row, 7.4 / 5.8 (4.9 / 5.2), 4 x 1024 x 768 (64) 6.0 / 5.1 (4.4 / 4.7); a gain from 64 tiles on,
//     below none (1 x 1024 x 768 5.2 / 4.9 (4.3 / 4.6)); from 9 rows on also below (12 rows 5.9 / 5.1 (5.0 / 4.8)).
//   - 16-bit: it splits K by four, and a chip full of tiles is what the narrow ones need, with loads past the caches (stream_b) or K beyond 512: 128 x 2048 x 768,
//     32 of the groups with a row (1024 tiles), 20.9 / 18.0, 16 (512) 12.2 / 11.0 and 8.0 / 7.8, 128 x 1536 x 2048 16 with a row (384) 21.7 / 22.1; weights that stay, and those
//     of three layers in turn: 16 x 2560 x 384 2 rows 8.0 / 9.4 and 7.7 / 8.4, 32 x 2048 x 512 4 rows 13.6 / 15.8 and 12.5 / 12.3, 32 x 1536 x 768 15.6 / 15.9 and 14.1 / 13.2, x 1024
//     20.3 / 19.5 and 19.0 / 17.0.
//     From 9 rows on its passes of 16 or 32 rows read the weights of uneven groups again: 16 x 1536 x 1024 12 rows 13.5 / 13.3 and 12.5 / 10.8, 8 x 1024 x 2048 (128)
//     11.4 / 11.1 and 10.1 / 8.6; with short K or few tiles from 13 on: 8 x 1024 x 768 12 rows 6.0 / 6.5 and 5.6 / 5.7, 4 x 1024 x 1024 (64) 12 rows 1.01 - 1.06 of its time, 20 rows
//     8.4 / 7.7 and 9.2 / 6.9, 64 x 2048 x 384 12 rows 21.5 / 22.2.
constexpr int kNarrowStages = 6;
inline int64_t narrow_tiles(const GemmArgs& g) { return (g.M < g.groups ? g.M : g.groups) * (g.N / 64); }   // columns of tiles in all groups that can have rows
inline bool narrow_fits(const GemmArgs& g) {
  const int eb = g.fp8 ? 1 : 2;
  if (g.b_kstep != 128 || g.b_tpb_shift || g.b_blk_stride != 256 * g.ldb || g.K * eb % 128 || g.K * eb / 128 < kNarrowStages || g.N % 64 || g.N / 64 > 2048) return false;
  if (g.groups > 1024) return false;
  if (g.fp8) return g.K >= 1024 || 4 * narrow_tiles(g) >= cu_count() || g.M > 8 * (int64_t)g.groups;
  if (narrow_tiles(g) > 2 * cu_count() && (g.stream_b || g.K > 512)) return true;
  return g.M > 64 && g.M > (g.K > 768 && 2 * narrow_tiles(g) >= cu_count() ? 8 : 12) * (int64_t)g.groups;
}
// Rows of a narrow tile, by the rows per group on average.  us, 16 / 32 / 64 rows: fp16 64 x 2816 x 2048 at 1 row 71 / 65 / 67, at 12 134 / 123 / 118,
// at 16 151 / 129 / 131, at 24 181 / 148 / 144; fp8 at 4 rows 53 / 54 / 57, at 8 59 / 57 / 58, at 16 70 / 64 / 61.  With rows of B a multiple of 4 KiB apart (one K-tile of
// all of them lies on a few of the memory's channels) and a chip full of tiles the two waves of a 16-row tile fall behind: fp8 16 x 2048 x 4096 at 4 rows
// 30.3 / 25.9, 64 x 1024 x 4096 54.6 / 46.0 (streaming kernel 50.6), 32 x 1024 x 8192 54.5 / 46.6; with fewer tiles they do not: 12 x 2048 x 4096 22.2 / 23.4, 2 x 2048 x 8192
// 17.1 / 17.7, and with one row per group on average, drawn, a third of the groups have none: 16 x 2048 x 4096 17.6 / 18.7, 64 x 1024 x 4096 38.4 / 32.7.
inline int narrow_rows(const GemmArgs& g) {
  const int64_t G = g.groups;
  const bool behind = g.ldb % 4096 == 0 && narrow_tiles(g) >= (g.M >= 2 * G ? 2 : 4) * cu_count();
  if (g.fp8 && g.M <= 4 * G && !behind) return 16;
  return g.M <= (g.fp8 ? 12 : 16) * G ? 32 : 64;
}

// Rows of a tile of the fused pair: what its two problems ask for (128 or 256, the same for both: grouped_pair_fusable), or, where both leave it to
// the library (left: no kernel asked for, and no threshold set for experiments), 192 for 177 to 192 rows per group on average and at least one and three
// quarter columns of tiles, 256 wide, per compute unit in either product (all groups).  The host knows the average, not the sizes, and the best height goes by the sizes: a group
// of 129 to 192 rows is one row block of 192 or two of 128, one of 193 to 256 two of either.  So 192 is taken only where it was not slower whatever the sizes; time on 192 rows
// over that on 128, fp16, groups drawn around the average with weights exp(N(0, 1/2)) (three draws) / all equal / a quarter of the rows in one group, the others equal:
//   - 180 rows per group (experts x hidden x intermediate): 128 x 2048 x 768 0.99 / 0.86 / 0.71, 256 x 2048 x 512 0.96 / 0.81 / 0.67, 64 x 2048 x 1024 0.97 / 0.82 / 0.75, 60 x 2048 x 1408 0.92 / 0.81 /
//     0.83, 128 x 4096 x 1536 0.99 / 0.81 / 0.57, 160 x 5120 x 1536 0.95 / 0.83 / 0.76; at 192 0.96 / 0.85 / 0.78, 0.96 / 0.84 / 0.66, 0.93 / 0.85 / 0.79, 0.91 / 0.80 / 0.83,
//     0.99 / 0.80 / 0.57, 1.01 / 0.82 / 0.79.
//   - fewer rows: with a quarter of them in one group the others have at most 128: at 150 1.05 / 0.99 / 1.08 / 1.07 / 1.06 / 1.00 (the same six).
//   - more rows: equal groups have two row blocks either way.  At 200 128 x 2048 x 768 0.94 / 1.34 / 0.77, 64 x 2048 x 1024 0.83 / 1.23 / 0.78, 160 x 5120 x 1536 1.03 / 1.47 / 0.74; at 256 0.95 / 1.15 / 1.28, 1.01 / 1.15 /
//     1.21, 1.03 / 1.41 / 1.36; at 320 0.95 / 0.90 / 1.17, 1.00 / 0.94 / 1.05, 1.00 / 1.02 / 1.33.  (256 rows, at 320: 1.01 / 1.10 / 0.87, 1.02 / 1.13 / 0.84, 1.01 / 1.21 / 0.81.)
//   - fewer tiles: whole rounds decide.  At 180 64 x 2048 x 768 (384 columns of tiles, 512) 1.05 / 0.92 / 0.82, 16 x 4096 x 2048 (256 columns of tiles in both products) 1.12 / 0.84 / 0.82, 64 x 1024 x 512 (256) 1.13 / 0.83 / 0.97, 8 x 4096 x 1792 (112, 128) 1.11 / 1.17 / 0.95, 8 x 2048 x 1024 (64)
//     1.11 / 1.18 / 1.09, 32 x 2048 x 768 (192, 256) 1.13 / 0.81 / 0.86, 8 x 4096 x 14336 (896, 128) 1.05 / 1.07 / 0.73.
inline int pair_tile_rows(const GemmArgs& g1, const GemmArgs& g2, bool left) {
  const int rows = grouped_tile_rows(g1.M, g1.groups, g1.tile_m);
  if (!left || rows != 128 || grouped_tile128_rows().set) return rows;
  const int64_t G = g1.groups, columns = G * (g1.grid_n < g2.grid_n ? g1.grid_n : g2.grid_n);
  return g1.M > 176 * G && g1.M <= 192 * G && 4 * columns >= 7 * (int64_t)cu_count() ? 192 : 128;
}
// Whether two planned grouped problems (the second reading what the first writes) can run as one launch: both on
// the chained tile pipeline, asking for the same tile height, and few enough tiles in the worst case that one workgroup per
// compute unit holds them all (a wave keeps 64 per GEMM) -- the workgroups must all be resident for the waits to end.  (Judged on the height
// asked for: pair_tile_rows takes none lower.)
inline bool grouped_pair_fusable(const GemmArgs& g1, const GemmArgs& g2) {
  const int cus = cu_count();
  const int tm = grouped_tile_rows(g1.M, g1.groups, g1.tile_m);
  if (g1.fp8 || g2.fp8 || g1.f16 != g2.f16 || g1.M != g2.M || g1.groups != g2.groups || !g1.gated || g2.gated || cus % 8) return false;
  if (tm != grouped_tile_rows(g2.M, g2.groups, g2.tile_m)) return false;
  for (const GemmArgs* g : {&g1, &g2}) {
    const int nk = (int)(g->K / 64);
    if (nk % 2 || nk < 4) return false;
    if ((g->M / tm + g->groups) * (int64_t)g->grid_n > 64 * (int64_t)cus) return false;
  }
  return true;
}

}  // namespace axe
