// The tile table of the grouped tile kernels (device code only): which tiles a workgroup owns, worked out on the
// device from the group offsets -- no scratch memory, no host knowledge of the group sizes.
#pragma once
#include <hip/hip_runtime.h>

#include "device_types.h"

namespace axe {

// Tiles of a grouped problem, counted group after group: group e has ceil(rows_e / TM) x grid_n of them
// (row blocks fastest).  Lane t of the calling wave receives the workgroup's t-th tile: its first row, its
// number of rows (0: no such tile), its tile column and its group.  Workgroup ids are dealt round-robin
// to the 8 XCDs, so XCD x takes the x-th eighth of the tile sequence and its 32 workgroups walk it side
// by side: neighbours in the sequence share A rows (same group and row block) or a B panel in that
// XCD's L2.  The offsets are clamped to [0, M], so that whatever they hold no access leaves the buffers.
// t_desc packs rows (bits 0..8), tile column (9..19) and group (20..31): the host admits at most 4096
// groups and 2048 tile columns.
__device__ __forceinline__ int desc_rows(int d) { return d & 511; }
__device__ __forceinline__ int desc_tn(int d) { return (d >> 9) & 2047; }
__device__ __forceinline__ int desc_group(int d) { return (int)((unsigned)d >> 20); }
// Inclusive prefix sum over the 64 lanes (row shifts inside 16 lanes, then two broadcasts of the rows before).
__device__ __forceinline__ int wave_prefix_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}
// Returns whether the weights are best loaded past the caches (kOnce): the host says so by their size, and at least three quarters
// of the tiles are the only row block of their group, so that no other tile reads their rows of B.  MoE layer of 128 experts, us, through the
// caches -> past them: fp16 256 / 512 / 1024 tokens 221 -> 199 / 232 -> 211 / 273 -> 254, E8M0 120 -> 107 / 128 -> 114 / 157 -> 143; with half of the
// rows in one group 259 -> 250 (fp16, 512 tokens).  Everywhere instead: 2048 / 4096 tokens 323 -> 371 / 444 -> 547 (40 % and more of the groups have a
// second row block, whose tile then reads the weights from memory again).
// What bounds the table: latency, before a workgroup's first load can be issued.  So: the offsets of the first 128 groups are
// fetched once, both halves at the same time, and every lane finds its tile's group by bisecting the prefix sums across lanes (six
// permutes), not by looking at the groups one after the other.  128 groups: about 10 us per launch less (an MoE layer of two products, us, before ->
// now: fp16 512 / 4096 tokens 252 -> 231 / 441 -> 423, fp8 with fp32 scales 1024 tokens 184 -> 159, E8M0 codes 256 tokens 146 -> 120).
template <int TM, bool ONE = false>                               // rows of a tile; ONE: a single group of all M rows, no offsets array
__device__ __forceinline__ bool group_tiles(const GemmArgs& g, int lane, int& t_row0, int& t_desc) {
  const int G = g.groups, M = (int)g.M, gn = g.grid_n;
  const int* __restrict__ off = g.group_rows;
  struct Chunk {
    int r0, rows, incl;                                            // a group per lane: first row, rows, inclusive prefix sum of tiles
  };
  auto fetch = [&](int g0, int& a, int& b) __attribute__((always_inline)) {
    const int gi = g0 + lane;
    a = 0, b = 0;
    if constexpr (ONE) {
      if (gi == 0) b = M;
    } else if (gi < G) {
      a = off[gi], b = off[gi + 1];
    }
  };
  auto blocks = [&](int rows) __attribute__((always_inline)) -> int { return (rows + TM - 1) / TM; };
  auto chunk = [&](int a, int b) __attribute__((always_inline)) -> Chunk {
    a = a < 0 ? 0 : (a > M ? M : a);
    b = b < 0 ? 0 : (b > M ? M : b);
    Chunk c;
    c.r0 = a;
    c.rows = b > a ? b - a : 0;
    c.incl = wave_prefix_sum(blocks(c.rows) * gn);
    return c;
  };
  int a0, b0, a1 = 0, b1 = 0;
  fetch(0, a0, b0);
  if (!ONE && G > 64) fetch(64, a1, b1);
  const Chunk c0 = chunk(a0, b0), c1 = chunk(a1, b1);
  int total = __builtin_amdgcn_readlane(c0.incl, 63) + __builtin_amdgcn_readlane(c1.incl, 63);
  auto single = [&](const Chunk& c) __attribute__((always_inline)) -> int { return __popcll(__ballot(c.rows > 0 && c.rows <= TM)); };
  int singles = single(c0) + single(c1);                           // groups of one row block
  for (int g0 = 128; g0 < G; g0 += 64) {
    fetch(g0, a0, b0);
    const Chunk c = chunk(a0, b0);
    total += __builtin_amdgcn_readlane(c.incl, 63), singles += single(c);
  }
  const bool once = g.stream_b && 4 * (int64_t)singles * gn >= 3 * (int64_t)total;
  const int per = (total + 7) >> 3;                                // tiles per XCD
  const int s = (int)(blockIdx.x >> 3) + lane * (int)(gridDim.x >> 3);
  const int u = (int)(blockIdx.x & 7) * per + s;                   // position of this lane's tile in the sequence
  const bool valid = s < per && u < total;
  int f_local = 0, f_rows = 0, f_r0 = 0, f_group = 0, base = 0;
  auto find = [&](const Chunk& c, int g0) __attribute__((always_inline)) {
    const int last = __builtin_amdgcn_readlane(c.incl, 63), at = u - base;
    int l = 0;                                                     // groups whose tiles all lie before this lane's
#pragma unroll
    for (int d = 32; d; d >>= 1)
      if (__shfl(c.incl, l + d - 1, 64) <= at) l += d;
    const int rows = __shfl(c.rows, l, 64), r0 = __shfl(c.r0, l, 64), incl = __shfl(c.incl, l, 64);
    if (valid && at >= 0 && at < last) f_local = at - (incl - blocks(rows) * gn), f_rows = rows, f_r0 = r0, f_group = g0 + l;
    base += last;
  };
  find(c0, 0);
  if (!ONE && G > 64) find(c1, 64);
  for (int g0 = 128; g0 < G; g0 += 64) {
    fetch(g0, a0, b0);
    find(chunk(a0, b0), g0);
  }
  // inside a group the row blocks run fastest: the tiles that read one B panel are neighbours in the
  // sequence (they run side by side on one XCD and the second reads the panel from that L2), and the
  // tiles that read one block of A rows are only a group's few row blocks apart
  const int gm = (f_rows + TM - 1) / TM;                           // row blocks of the group (0: the lane found no tile)
  const int tn = gm ? f_local / gm : 0;
  const int tm = f_local - tn * gm;
  t_row0 = f_r0 + tm * TM;
  const int left = f_rows - tm * TM;
  t_desc = (left < TM ? left : TM) | (tn << 9) | (f_group << 20);
  return once;
}

}  // namespace axe
