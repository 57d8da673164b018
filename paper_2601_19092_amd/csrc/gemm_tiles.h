// GEMM on small and medium tiles for gfx950 (device code): one kernel body, its tile, wave grid and K split template
// parameters (tile_family.h).  It serves what the 256-row kernels are too coarse for: a decode step's handful of rows,
// prefill chunks, edges that fill no large tile, and fp8 with scales the matrix cores' scale path cannot carry.
//
// What bounds it.  A K-step of a TM x TN tile moves (TM + TN) x 128 bytes for TM x TN x 128 bytes' worth of products; at the 21 - 25
// TB/s the L2s deliver (about 86 GB/s per CU) a 128 x 128 tile's K-step takes 370 ns, of which the matrix cores need 240.  Hence
// tiles as large as the problem can fill the chip with, every load instruction 8 rows of whole 128-byte lines straight into
// LDS (buffer_load ... lds: no registers, no ds_write), and a ring deep enough to keep 96 - 128 KiB in flight per CU.  What it
// reaches is less: 50 - 62 GB/s per CU over a whole launch of 128 x 128 tiles, 73 - 87 inside long K loops (matrix cores 46 % and 41 % busy in
// the two shapes below).  Builds with parts taken out, clocks of a K-step at 2.4 GHz, fp16 2000 x 2000 x 2048 / fp8 with row scales 1000 x 3584 x 8192 / bf16 1024 x
// 3584 x 8192: all of it 1380 / 1380 / 1120, loads and barriers alone 940 / 900 / 800, LDS reads alone (96 KiB in eight waves of 32 x 64) 680 / 590 / 620, matrix work with the
// fold alone 710 / 1060 / 660.  So no part is the whole of it; they overlap to about two thirds.
//
// Tile movements (tile_maps.h, the image of the 256-row kernels):
//   HBM -> LDS  : pieces of 8 rows x 128 bytes, one wave instruction each; the XOR swizzle is applied on the global side.
//   LDS layout  : a stage holds one K-tile (128 bytes of K) of TM rows of A and TN rows of B for each of the WK wave
//                 groups; 16-byte chunk c of row r at chunk position c ^ ((r >> 1) & 7).
//   LDS -> VGPR : lane l reads row l % 16 of a fragment, chunks l / 16 and l / 16 + 4 (16-bit inputs: two MFMAs
//                 16x16x32; fp8: the 32 bytes of one MFMA 16x16x128).
//   MFMA        : operands swapped (B rows first), so a lane's accumulator fragment holds 4 consecutive columns of a row.
//
// Pipeline.  The loads of stage s + NST are issued while stage s is multiplied; the wait at the head of a step, for stage
// s + 1, is counted (the loads of the NST - 2 stages after it stay in flight) and followed by one workgroup barrier -- or none
// when a wave group is a single wave, which then reads only what it loaded itself.  Chunks past K, rows past the
// operand's end and stages past the last K-tile get an offset no descriptor reaches: they load as zeros at no traffic,
// and the counts stay the same.
//   The fragments of stage s + 1 are read before stage s is multiplied: two waves per SIMD alone do not cover the LDS
// latency (128 x 128, bf16 2048^3: 20.8 us without, 18.5 with).  Eight waves of 32 x 64 on a 128 x 128 tile beat four of
// 64 x 64 (28 us), two K groups of 64 x 64 waves (24.7), sixteen of 32 x 32 (20.3) and two workgroups per CU with two stages
// each (27.6 there, level on 512 tiles).
//
// Measured, us, against the 64 x 64 kernel that served these problems: bf16 16 x 3584 x 8192 91.5 -> 11.4 (58.9 MB, 5.2 TB/s),
// 64 x 3584 x 8192 94 -> 15, 512 x 3584 x 8192 101 -> 40, fp16 2000 x 2000 x 2048 39 -> 19 - 21 (770 - 860 TFLOP/s), fp8 with one fp32 scale per
// row 1000 x 3584 x 8192 365 -> 37 - 39 (1500 - 1590 TFLOP/s), fp8 E8M0 256 x 512 x 6400 105 -> 7.6; and against the large tile: fp8
// 1024 x 3584 x 8192 76 -> 36, bf16 2048 x 4096 x 2048 40 -> 34.
//
// Scales (fp8).  A K-tile is one 128-deep scale block: its product is formed alone and folded into the sum on the vector
// ALU with the row's scale times the column block's (fp32, or E8M0 codes built as 2^(their sum - 254)).  Two codes may
// add up to a power of two that no float holds, where the product is zero or small, so they are scale operands of the matrix
// instruction.  The same bits as factors give, and as fast in most tiles (us, factors / codes: 512 x 3584 x 8192 25.1 / 25.1, 300 x 1024 x 1024
// 6.0 / 6.0, but 2048 x 4096 x 8192 65.4 / 68.7); the 128 x 128 tile, where they are not (1024 x 3584 x 8192 35.8 / 37.9),
// multiplies by factors up to the first trip whose codes have none, and runs a second K loop from there (35.1; the largest tile has no
// registers for two loops, in the others they cost 2 - 9 %).  Adding in place too, 34.2 here, gives sums that are less exact.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_types.h"
#include "gemm_common.h"
#include "grouped_tiles.h"
#include "kernels.h"
#include "tile_family.h"
#include "tile_maps.h"

namespace axe {
namespace tiles {

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(3))) uint8_t* lds_u8;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
// rows of C start at any element (odd N): global memory takes the vector there, four element stores cost four times as much
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));

template <int DT>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  if constexpr (DT == 1) {
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    const f16x2 v = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, v);
  } else {
    return pack_bf16(lo, hi);
  }
}

// A descriptor from values that are the same in every lane.  Said explicitly: a grouped launch reads them out of its table, and where the compiler
// keeps one in a vector register it wraps every load in a loop over the lanes' values (fp8 layer with fp32 scales, us: 512 tokens 124 -> 119, 4096 tokens 312 -> 297).
template <bool SAY>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const uint8_t* p, int bytes) {
  if constexpr (SAY) {
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    p = (const uint8_t*)((uint64_t)hi << 32 | lo);
    bytes = __builtin_amdgcn_readfirstlane(bytes);
  }
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, 0x00020000);
}

template <int N>
__device__ __forceinline__ void wait_loads() {                     // all but this wave's last N loads have landed; its LDS reads are done
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// DT: 0 bf16, 1 fp16, 2 fp8 e4m3.  SC (fp8): 0 unscaled, 1 fp32 scales, 2 E8M0 codes, 3 E8M0 codes multiplied as floats.
// GRP: 0 dense; 1, 2 grouped (A's scales one per row), 2 with the gated epilogue.  A grouped launch finds its workgroup's
// tiles on the device (grouped_tiles.h) and walks them one after the other.  ONCE: B is loaded past the caches.  PLACED: reads and
// loads have their places between the matrix instructions (launch_member).
// Where AXE_TILES_BODY is defined this is a function, for kernels with more than one body (which hand it the workgroup's LDS and the table).  Not
// everywhere: as a function inside a kernel it compiles to other code (a decode step of 16 rows 11.41 -> 11.46 us).
template <int DT, int SC, int TM, int TN, int WM, int WN, int WK, int NST, int GRP = 0, bool ONCE = false, bool PLACED = false>
#ifdef AXE_TILES_BODY
__device__ __forceinline__ void gemm_tiles_body(GemmArgs g, lds_u8 lds3, int t_row0, int t_desc) {
#else
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm_tiles_kernel(GemmArgs g) {
#endif
  constexpr int EB = DT == 2 ? 1 : 2;
  constexpr int kRow = maps::kLargeRowBytes;
  constexpr int NG = WM * WN;                                      // waves of a group
  constexpr int MF = TM / WM / 16, NF = TN / WN / 16;              // fragments of a wave
  constexpr int PA = TM / 8 / NG, PB = TN / 8 / NG;                // pieces of A and of B per wave and stage
  constexpr int kLoads = PA + PB;
  constexpr int kGroup = (TM + TN) * kRow, kStage = WK * kGroup;   // bytes of a group's K-tile, of a stage
  constexpr int U = SC ? 4 : 2;                                    // stages per trip of the main loop
  constexpr int NB = GRP == 2 ? 2 : 1;                             // column blocks of B's scales that a wave needs
  static_assert(TM % (16 * WM) == 0 && TN % (16 * WN) == 0 && (TM / 8) % NG == 0 && (TN / 8) % NG == 0, "whole fragments and pieces");
  static_assert(NST * kStage <= 160 * 1024 && (WK - 1) * TM * TN * 4 <= NST * kStage, "the ring, and then the partial sums, fit LDS");
  static_assert((NST - 1) * kLoads <= 63, "the counted wait");
#ifndef AXE_TILES_BODY
  __shared__ __attribute__((aligned(1024))) uint8_t lds_mem[NST * kStage];
  const lds_u8 lds3 = (lds_u8)lds_mem;
  if (GRP != 0 && g.clear && blockIdx.x == 0 && threadIdx.x == 0) *g.clear = 0;
#endif
  // the arguments in one fetch: left alone they come one by one, where each is first used, and every fetch is waited for
  if constexpr (GRP == 0) {
    asm volatile("" ::"s"(g.A), "s"(g.B), "s"(g.C), "s"(g.M), "s"(g.N), "s"(g.K), "s"(g.lda), "s"(g.ldb), "s"(g.ldc));
    asm volatile("" ::"s"(g.grid_m), "s"(g.grid_n), "s"(g.map.div_group), "s"(g.map.div_last), "s"(g.map.deal), "s"(g.map.turns), "s"(g.c_vec), "s"(g.out_bf16));
    if constexpr (SC != 0) asm volatile("" ::"s"(g.scale_a), "s"(g.scale_b), "s"(g.scale_a_rows), "s"(g.nkb));
  }
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int kpart = w / NG, wg = w % NG;                           // group, wave inside the group
  const int wm = wg / WN, wn = wg % WN;

  const int kbytes = (int)(g.K * EB);                              // bytes of K per row
  const int nk = (kbytes + kRow - 1) / kRow;                       // K-tiles
  // stages, whole trips of them; grouped: a last trip may be half a one (the branch costs a dense launch, whose K loop is its
  // whole time, 3 %).  Stages past the last K-tile multiply zeros.
  constexpr bool kHalfTrip = GRP != 0 && U == 4;
  constexpr int kWhole = kHalfTrip ? 2 : U;
  // A trip's scales are worked out at the end of the trip before, in either of its ends: at a common place the compiler's own wait for them
  // would allow no more loads in flight than follow them in half a trip.  (The 128-row tile has no registers for that, and a ring no longer.)
  constexpr bool kSpreadAhead = kHalfTrip && NST > 4;
  const int ns = ((nk + WK - 1) / WK + kWhole - 1) / kWhole * kWhole;
  const int a_pitch = (int)(g.lda * EB), b_pitch = (int)(g.ldb * EB);
  // ---- HBM -> LDS: this wave's pieces of a K-tile: of A, then of B
  constexpr int kOutside = 0x7fff0000;                             // past the end of every descriptor (the host keeps them below 2^30 bytes)
  const int lr = lane / maps::kLargeChunks, lp = lane % maps::kLargeChunks;
  int kchunk[kLoads];                                              // offset of the lane's chunk inside its row
#pragma unroll
  for (int i = 0; i < kLoads; ++i)
    kchunk[i] = maps::lds_chunk_pos(maps::piece_row(wg, i < PA ? i : i - PA, lr, NG), lp, maps::kLargeChunks) * maps::kChunkBytes;
  int voff[kLoads];                                                // offset of the lane's chunk in the operand
#pragma unroll
  for (int i = 0; i < kLoads; ++i) voff[i] = maps::piece_row(wg, i < PA ? i : i - PA, lr, NG) * (i < PA ? a_pitch : b_pitch) + kchunk[i];
  // The workgroup's tiles.  Dense: one, found from its id.  Grouped: found on the device, one per lane; the loads run on from
  // a tile's last stage into the next tile's first ones, so the load side, the scales and the matrix side each keep a
  // place of their own.
#ifndef AXE_TILES_BODY
  int t_row0 = 0, t_desc = 0;
  if constexpr (GRP != 0) group_tiles<TM>(g, lane, t_row0, t_desc);
#endif
  struct Place {
    int64_t m0, n0;
    int rows, cols, group;                                         // rows = 0: no such tile
  };
  auto place = [&](int t) __attribute__((always_inline)) -> Place {
    Place o;
    if constexpr (GRP != 0) {
      const int d = t < 64 ? __builtin_amdgcn_readlane(t_desc, t) : 0;
      o.rows = desc_rows(d), o.cols = TN, o.group = desc_group(d);
      o.m0 = __builtin_amdgcn_readlane(t_row0, t & 63), o.n0 = (int64_t)desc_tn(d) * TN;
    } else {
      const TileAt at = family_tile(blockIdx.x, g.grid_m, g.grid_n, g.map);
      const int tm = at.tm, tn = at.tn;
      o.m0 = (int64_t)tm * TM, o.n0 = (int64_t)tn * TN, o.group = 0;
      o.rows = g.M - o.m0 < TM ? (int)(g.M - o.m0) : TM, o.cols = g.N - o.n0 < TN ? (int)(g.N - o.n0) : TN;
    }
    return o;
  };
  Place here = place(0);                                           // the tile being multiplied
  if (here.rows == 0) return;                                      // (the whole workgroup: no barrier is left waiting)
  __amdgpu_buffer_rsrc_t ra, rb;                                   // the tile being loaded: rows past the end lie outside the descriptors
  int l_stage = 0, l_tile = 0, l_bytes = 0;
  auto load_from = [&](const Place& p) __attribute__((always_inline)) {
    l_stage = 0;
    l_bytes = p.rows ? kbytes : 0;
    // (no such tile: an empty descriptor -- (0 - 1) rows would wrap round to one that reaches everything)
    const int a_bytes = p.rows ? (p.rows - 1) * a_pitch + kbytes : 0;
    ra = uniform_rsrc<GRP != 0>((const uint8_t*)g.A + p.m0 * g.lda * EB, a_bytes);
    rb = uniform_rsrc<GRP != 0>((const uint8_t*)g.B + (p.group * g.ldg + p.n0 * g.ldb) * EB, (p.cols - 1) * b_pitch + kbytes);
  };
  load_from(here);
  auto issue = [&](int slot) __attribute__((always_inline)) {     // the load side's next stage
    const int kt = l_stage * WK + kpart;
    const int left = l_bytes - kt * kRow;                          // bytes of K from this K-tile on
    const lds_u8 base = lds3 + slot * kStage + kpart * kGroup;
    const int soff = left > 0 ? kt * kRow : 0;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const bool is_a = i < PA;
      const int off = kchunk[i] < left ? voff[i] : kOutside;
      const lds_ptr to = (lds_ptr)(base + (is_a ? 0 : TM * kRow) + maps::piece_row(wg, is_a ? i : i - PA, 0, NG) * kRow);
      if (is_a) __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, to, 16, off, soff, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, to, 16, off, soff, 0, ONCE ? kOnce : 0);
      AXE_PARANOID_WAIT();
    }
    ++l_stage;
    if (GRP != 0 && l_stage == ns) load_from(place(++l_tile));
  };

  // ---- LDS -> VGPR
  const int fr = lane % maps::kFrag, fq = lane / maps::kFrag;
  const int pos0 = maps::lds_chunk_pos(fr, maps::operand_chunk_fp8(0, fq), maps::kLargeChunks) * maps::kChunkBytes;
  const int pos1 = maps::lds_chunk_pos(fr, maps::operand_chunk_fp8(1, fq), maps::kLargeChunks) * maps::kChunkBytes;
  const int fa_off = kpart * kGroup + (wm * (TM / WM) + fr) * kRow, fb_off = kpart * kGroup + (TM + wn * (TN / WN) + fr) * kRow;
  auto read = [&](lds_u8 p) __attribute__((always_inline)) -> i32x4 { return *(__attribute__((address_space(3))) const i32x4*)p; };

  f32x4 acc[MF][NF];

  // ---- scales.  Lane (fr, fq) holds, for each of its fragment rows, the product of the row's and the column block's scale in
  //      the K-tile of stage s0 + fq; two swaps between lane groups hand every lane those of all four stages of a trip.
  //      One load per fragment row and one for the column block serve four stages; they are issued a trip ahead.
  //      With the gated epilogue the wave's gate and up columns lie in one column block each.
  constexpr int kScaleLoads = SC ? MF + NB : 0;
  constexpr int SB = SC >= 2 ? 1 : 4;                              // bytes of a stored scale
  const bool by_row = GRP != 0 || g.scale_a_rows == 1;
  int sa_off[SC ? MF : 1];
#pragma unroll
  for (int i = 0; i < (SC ? MF : 0); ++i) {
    const int r = wm * (TM / WM) + i * 16 + fr;                    // (rows past the end: any value, they are never stored)
    sa_off[i] = (by_row ? r : r / 128) * g.nkb * SB;
  }
  static_assert((TM <= 128 || TM % 128 == 0) && TN <= 128, "row blocks of scales start with a tile or inside one, a tile lies in one column block");
  uint32_t sa_raw[SC ? MF : 1], sb_raw[NB];
  __amdgpu_buffer_rsrc_t rsa, rsb[NB];
  auto scales_from = [&](const Place& p) __attribute__((always_inline)) {
    if constexpr (SC != 0) {
      const int64_t a0 = by_row ? p.m0 : p.m0 / 128;
      const int an = p.rows == 0 ? 1 : (by_row ? p.rows : (p.rows + 127) / 128);
      rsa = uniform_rsrc<GRP != 0>((const uint8_t*)g.scale_a + a0 * g.nkb * SB, an * g.nkb * SB);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        // gated: image rows n0 + wn TN / WN .. hold the logical gate columns from half of that on, and the up columns N / 2 further
        const int64_t col = GRP == 2 ? b * (g.N / 2) + (p.n0 + wn * (TN / WN)) / 2 : p.n0;
        const int64_t b0 = (GRP != 0 ? p.group * (g.N / 128) : 0) + col / 128;
        rsb[b] = uniform_rsrc<GRP != 0>((const uint8_t*)g.scale_b + b0 * g.nkb * SB, g.nkb * SB);
      }
    }
  };
  scales_from(here);
  auto fetch_scales = [&](int s0) __attribute__((always_inline)) {
    if constexpr (SC != 0) {
      asm volatile("" ::: "memory");                               // the waits below count these loads: they stay where they are
      const int kt = (s0 + fq) * WK + kpart;
      const int o = (kt < nk ? kt : nk - 1) * SB;
      auto load = [&](__amdgpu_buffer_rsrc_t r, int off) -> uint32_t {
        if constexpr (SC >= 2) return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
        else return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
      };
#pragma unroll
      for (int b = 0; b < NB; ++b) sb_raw[b] = load(rsb[b], o);
#pragma unroll
      for (int i = 0; i < MF; ++i) sa_raw[i] = load(rsa, sa_off[i] + o);
      asm volatile("" ::: "memory");
    }
  };
  float sc[NB][SC ? MF : 1][4];
  // the scales of a trip as factors; true: E8M0 codes among them whose power of two is no normal number
  auto spread_scales = [&](int s0) __attribute__((always_inline)) -> bool {
    bool far = false;
    if constexpr (SC != 0) {
      if constexpr (GRP != 0) {                                    // not before: the compiler's own wait for them would be stricter than the counted ones
#pragma unroll
        for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(sb_raw[b]));
#pragma unroll
        for (int i = 0; i < MF; ++i) asm volatile("" : "+v"(sa_raw[i]));
      }
      const bool in = (s0 + fq) * WK + kpart < nk;                 // stages past the last one multiply zeros by zero
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < MF; ++i) {
          uint32_t v;
          if constexpr (SC == 2) {
            v = (sa_raw[i] + sb_raw[b] - 127u) << 23;
            far = far || (in && sa_raw[i] + sb_raw[b] - 128u >= 254u);
          } else {
            const int up = SC == 3 ? 23 : 0;                       // a code as the exponent of a float
            v = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, sa_raw[i] << up) * __builtin_bit_cast(float, sb_raw[b] << up));
          }
          v = in ? v : 0u;
          const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
          const auto q0 = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
          const auto q2 = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
          sc[b][i][0] = __builtin_bit_cast(float, (uint32_t)q0[0]), sc[b][i][1] = __builtin_bit_cast(float, (uint32_t)q0[1]);
          sc[b][i][2] = __builtin_bit_cast(float, (uint32_t)q2[0]), sc[b][i][3] = __builtin_bit_cast(float, (uint32_t)q2[1]);
        }
    }
    if constexpr (SC == 2) return __ballot(far) != 0;
    else return false;
  };
  // the same as codes, a byte per stage of the trip (stages past the last one multiply zeros by one)
  uint32_t sa_codes[SC == 2 ? MF : 1], sb_codes = 0;
  auto spread_codes = [&](int s0) __attribute__((always_inline)) {
    if constexpr (SC == 2) {
      const bool in = (s0 + fq) * WK + kpart < nk;
      auto codes = [&](uint32_t raw) __attribute__((always_inline)) -> uint32_t {
        const uint32_t v = (in ? raw : 127u) << (8 * fq);
        const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        const uint32_t w = h[0] | h[1];
        const auto q = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        return q[0] | q[1];
      };
#pragma unroll
      for (int i = 0; i < MF; ++i) sa_codes[i] = codes(sa_raw[i]);
      sb_codes = codes(sb_raw[0]);
    }
  };
  // product of two fragments' K-tile times 2^(code - 127) of either, stage u of the trip
  auto scaled_product = [&](const i32x8& b, const i32x8& a, uint32_t a_codes, int u) __attribute__((always_inline)) -> f32x4 {
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    switch (u) {                                                   // (the byte is an immediate of the instruction)
      case 0: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, z, 0, 0, 0, (int)sb_codes, 0, (int)a_codes);
      case 1: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, z, 0, 0, 1, (int)sb_codes, 1, (int)a_codes);
      case 2: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, z, 0, 0, 2, (int)sb_codes, 2, (int)a_codes);
      default: return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, z, 0, 0, 3, (int)sb_codes, 3, (int)a_codes);
    }
  };

  struct Frags {
    i32x4 a[MF][2], b[NF][2];
  };
  auto read_frags = [&](Frags& f, int slot) __attribute__((always_inline)) {
    const lds_u8 base = lds3 + slot * kStage;
#pragma unroll
    for (int j = 0; j < NF; ++j) f.b[j][0] = read(base + fb_off + j * 16 * kRow + pos0), f.b[j][1] = read(base + fb_off + j * 16 * kRow + pos1);
#pragma unroll
    for (int i = 0; i < MF; ++i) f.a[i][0] = read(base + fa_off + i * 16 * kRow + pos0), f.a[i][1] = read(base + fa_off + i * 16 * kRow + pos1);
  };
  auto multiply = [&](const Frags& f, int u, auto far) __attribute__((always_inline)) {
    if constexpr (DT != 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
          for (int j = 0; j < NF; ++j)
            if constexpr (DT == 1) {
              typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, f.b[j][h]), __builtin_bit_cast(f16x8, f.a[i][h]), acc[i][j], 0, 0, 0);
            } else {
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.b[j][h]), __builtin_bit_cast(bf16x8, f.a[i][h]), acc[i][j], 0, 0, 0);
            }
    } else {
      auto wide = [](const i32x4* p) { return i32x8{p[0][0], p[0][1], p[0][2], p[0][3], p[1][0], p[1][1], p[1][2], p[1][3]}; };
#pragma unroll
      for (int i = 0; i < MF; ++i) {
        if constexpr (far) {
          f32x4 p[NF];
#pragma unroll
          for (int j = 0; j < NF; ++j) p[j] = scaled_product(wide(f.b[j]), wide(f.a[i]), sa_codes[i], u);
#pragma unroll
          for (int j = 0; j < NF; ++j) {
            acc[i][j] += p[j];
            // (in order where a group has K to itself: products waiting for their sums would spill in the largest tile and cost the
            //  128 x 64 one 2 - 4 %; the small ones are 2 % faster as the compiler likes it: 300 x 1024 x 1024 6.0 us, 6.2 in order)
            if constexpr (WK == 1) asm volatile("" : "+v"(acc[i][j]));
          }
        } else if constexpr (SC != 0) {
          f32x4 p[NF];
#pragma unroll
          for (int j = 0; j < NF; ++j)
            p[j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wide(f.b[j]), wide(f.a[i]), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = __builtin_fmaf(sc[NB == 2 ? j & 1 : 0][i][u], p[j][e], acc[i][j][e]);
        } else {
#pragma unroll
          for (int j = 0; j < NF; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wide(f.b[j]), wide(f.a[i]), acc[i][j], 0, 0, 0, 0, 0, 0);
        }
      }
    }
  };

  // ---- prologue: the first tile's first stages
  Frags f[2];
  fetch_scales(0);
#pragma unroll
  for (int s = 0; s < NST; ++s) issue(s);
  wait_loads<(NST - 1) * kLoads>();
  if constexpr (NG > 1) wg_barrier();
  AXE_PARANOID_SYNC();
  read_frags(f[0], 0);

  if constexpr (kSpreadAhead) spread_scales(0);
  int cur = 0;                                                     // slot of the stage whose fragments are in f[u & 1]
  for (int t = 1;; ++t) {
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr bool kCodesOnly = SC == 2 && MF * NF != 8;
  int s0 = 0;
  // stage u of the trip; far: E8M0 scales as codes.  (The loops over u stay outside: unrolled inside a lambda they are scheduled
  // otherwise, 1000 x 3584 x 8192 with row scales 39.3 -> 39.5 us.)
  auto stage = [&](int u, auto far) __attribute__((always_inline)) {
    // stage s + 1 has landed, everybody's reads of stage s are done: its slot takes stage s + NST.  (The scales fetched
    // at the head of the trip are younger than the stages up to s0 + NST - 1; whatever else is in flight only makes a
    // counted wait stricter.)
    if (u >= 1 && u <= NST - 2) wait_loads<(NST - 2) * kLoads + kScaleLoads>();
    else wait_loads<(NST - 2) * kLoads>();
    if constexpr (NG > 1) wg_barrier();
    AXE_PARANOID_SYNC();
    if constexpr (PLACED) __builtin_amdgcn_sched_barrier(0);
    const int nxt = cur + 1 == NST ? 0 : cur + 1;
    read_frags(f[(u + 1) & 1], nxt);
    if (u == 0) {
      const bool last = GRP != 0 && s0 + U >= ns;                // the next trip is the next tile's first
      if (last) scales_from(place(t));
      fetch_scales(last ? 0 : s0 + U);
    }
    issue(cur);
    multiply(f[u & 1], u, far);
    if constexpr (PLACED) {                                        // one matrix instruction, then its share of the reads and, after them, of the loads
      constexpr int kReads = (MF + NF) * 2, kProducts = MF * NF * (DT == 2 ? 1 : 2), kOthers = kReads + kLoads;
#pragma unroll
      for (int m = 0; m < kProducts; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int k = m * kOthers / kProducts; k < (m + 1) * kOthers / kProducts; ++k)
          if (k < kReads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          else __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  };
  if constexpr (kSpreadAhead) {
    for (; s0 < ns; s0 += U) {
      stage(0, std::false_type{}), stage(1, std::false_type{});
      if (s0 + 2 >= ns) {
        spread_scales(0);
        break;
      }
      stage(2, std::false_type{}), stage(3, std::false_type{});
      spread_scales(s0 + U >= ns ? 0 : s0 + U);
    }
  } else if constexpr (!kCodesOnly) {
    for (; s0 < ns; s0 += U) {
      if (spread_scales(s0)) break;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (kHalfTrip && u == 2 && s0 + 2 >= ns) break;
        stage(u, std::false_type{});
      }
    }
  }
  if constexpr (SC == 2)
    for (; s0 < ns; s0 += U) {
      spread_codes(s0);
#pragma unroll
      for (int u = 0; u < U; ++u) stage(u, std::true_type{});
    }

  // ---- the groups' sums meet in LDS: group 0 adds them in the order of the groups
  if constexpr (WK > 1) {
    wait_loads<0>();                                               // (the zeros of stages past the end have landed, too)
    wg_barrier();
    typedef __attribute__((address_space(3))) f32x4* lds_f32x4;
    auto slot = [&](int part, int i, int j) -> lds_f32x4 {
      return (lds_f32x4)(lds3 + (((part - 1) * NG + wg) * MF * NF + i * NF + j) * 1024 + lane * 16);
    };
    if (kpart > 0) {
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) *slot(kpart, i, j) = acc[i][j];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();
    if (kpart > 0) return;
#pragma unroll
    for (int part = 1; part < WK; ++part)
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] += *slot(part, i, j);
  }

  // ---- VGPR -> HBM: lane holds C[m][n .. n + 3]
  // Through a descriptor of the tile's part of C where the host says so (c_vec): rows past the end lie outside it, columns past the end get an
  // offset that does, and a fragment's place is one addition and an immediate.  The rows go into the offset that is checked against the
  // descriptor's end, not into the scalar one, which is documented as left out of that check.
  if constexpr (GRP == 0) {
    if (g.c_vec) {
      const int cb = g.out_bf16 ? 2 : 4, c_pitch = (int)g.ldc * cb;
      const __amdgpu_buffer_rsrc_t rc =
          __builtin_amdgcn_make_buffer_rsrc((uint8_t*)g.C + (here.m0 * g.ldc + here.n0) * cb, 0, (here.rows - 1) * c_pitch + here.cols * cb, 0x00020000);
      const int col = wn * (TN / WN) + maps::kAccCols * fq, at = (wm * (TM / WM) + fr) * c_pitch + col * cb;
#pragma unroll
      for (int i = 0; i < MF; ++i) {
        const int row_at = at + i * 16 * c_pitch;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          const int off = col + j * 16 < here.cols ? row_at : kOutside;
          if (g.out_bf16) {
            const u32x2 d = {pack2<DT>(acc[i][j][0], acc[i][j][1]), pack2<DT>(acc[i][j][2], acc[i][j][3])};
            __builtin_amdgcn_raw_buffer_store_b64(d, rc, off + j * 32, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), rc, off + j * 64, 0, 0);
          }
        }
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < MF; ++i) {
    const int r = wm * (TM / WM) + i * 16 + fr;
    if (r >= here.rows) continue;
    const int64_t m = here.m0 + r;
    if constexpr (GRP == 2) {                                      // fragments 2 p and 2 p + 1: gate and up of the same 16 outputs
#pragma unroll
      for (int p = 0; p < NF / 2; ++p) {
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gate = acc[i][2 * p][e], up = acc[i][2 * p + 1][e];
          h[e] = gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up;
        }
        uint16_t* C = (uint16_t*)g.C + m * g.ldc + (here.n0 + wn * (TN / WN)) / 2 + p * 16 + maps::kAccCols * fq;
        *(u32x2*)C = u32x2{pack2<DT>(h[0], h[1]), pack2<DT>(h[2], h[3])};
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int64_t n = here.n0 + wn * (TN / WN) + j * 16 + maps::kAccCols * fq;
      if (g.out_bf16) {
        uint16_t* C = (uint16_t*)g.C + m * g.ldc + n;
        const u32x2 d = {pack2<DT>(acc[i][j][0], acc[i][j][1]), pack2<DT>(acc[i][j][2], acc[i][j][3])};
        if (n + 3 < g.N) {
          *(u32x2_any*)C = d;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < g.N) C[e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
        }
      } else {
        float* C = (float*)g.C + m * g.ldc + n;
        if (n + 3 < g.N) {
          *(f32x4_any*)C = acc[i][j];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < g.N) C[e] = acc[i][j][e];
        }
      }
    }
  }
  if constexpr (GRP == 0) return;
  here = place(t);
  if (here.rows == 0) return;
  }
}

#ifndef AXE_TILES_BODY
template <int DT, int SC, int F>
hipError_t launch_member(const GemmArgs& g, hipStream_t s) {
  constexpr TileShape t = kTileFamily[F];
  auto launch = [&](auto placed) {
    hipLaunchKernelGGL((gemm_tiles_kernel<DT, SC, t.tm, t.tn, t.wm, t.wn, t.wk, t.nst, 0, false, decltype(placed)::value>), dim3((unsigned)(g.grid_m * g.grid_n)),
                       dim3(64 * t.wm * t.wn * t.wk), 0, s, g);
    return hipGetLastError();
  };
  constexpr bool shortest = family_placed(F, SC, 0), longest = family_placed(F, SC, INT64_MAX);
  if constexpr (shortest != longest)
    if (!family_placed(F, SC, g.K)) return launch(std::false_type{});
  return launch(std::bool_constant<longest>{});
}

template <int DT, int SC>
hipError_t launch_family(int member, const GemmArgs& g, hipStream_t s) {
  switch (member) {
    case 0: return launch_member<DT, SC, 0>(g, s);
    case 1: return launch_member<DT, SC, 1>(g, s);
    case 2: return launch_member<DT, SC, 2>(g, s);
    case 3: return launch_member<DT, SC, 3>(g, s);
    case 4: return launch_member<DT, SC, 4>(g, s);
    case 5: return launch_member<DT, SC, 5>(g, s);
    case 6: return launch_member<DT, SC, 6>(g, s);
    case 7: return launch_member<DT, SC, 7>(g, s);
    case 8: return launch_member<DT, SC, 8>(g, s);
    default: return hipErrorInvalidValue;
  }
  static_assert(kTileFamilySize == 9, "one case per member");
}
#endif

}  // namespace tiles
}  // namespace axe
