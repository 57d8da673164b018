// Plain-data descriptors handed from the host layer to the kernels by value (kernel arguments).
#pragma once
#include <stdint.h>

#include "tile_family.h"

namespace axe {

constexpr int kMaxD = 16;
constexpr int kMaxR = 8;
constexpr int kMaxAxes = 8;
constexpr int kMaxJoint = 24;   // common refinement of two D lists can be longer than either

// XOR stage: y = x ^ (((x >> shift) & mask) << base); mask == 0 disables it.
struct Swz {
  int32_t mask, base, shift;
};

// Division of 31-bit numbers by a fixed d > 1 as a multiplication: with 2^(s-1) < d <= 2^s and m = floor(2^(31+s) / d) + 1 (below
// 2^32), floor(n m / 2^(31+s)) = floor(n / d) for every n < 2^31, since m d - 2^(31+s) <= 2^s.  Two instructions, where a
// division by a run-time number takes some 25 on the vector ALU.
struct Div31 {
  uint32_t mul;                // 0: not prepared
  int32_t shift;               // s - 1
};
inline Div31 div31_by(int64_t d) {
  if (d < 2 || d >= (int64_t(1) << 31)) return Div31{0, 0};
  int s = 0;
  while ((int64_t(1) << s) < d) ++s;
  return Div31{(uint32_t)(((uint64_t(1) << (31 + s)) / (uint64_t)d) + 1), s - 1};
}
#if defined(__HIPCC__)
__host__ __device__
#endif
inline uint32_t div31(uint32_t n, Div31 d) { return (uint32_t)(((uint64_t)n * d.mul) >> 32) >> d.shift; }

// Full layout for axe_layout_eval (all axes kept).
struct EvalDesc {
  int32_t n_d, n_r, n_axes;
  int32_t use32;               // E_D < 2^31: digit arithmetic in 32 bits
  int32_t shift[kMaxD];        // log2(ext) when ext is a power of two, else -1
  Div31 div[kMaxD];            // otherwise, when use32
  int64_t ext[kMaxD], str[kMaxD];
  int32_t axis[kMaxD];
  int64_t rext[kMaxR], rstr[kMaxR];
  int32_t raxis[kMaxR];
  int64_t off[kMaxAxes];
  int32_t swz_axis;
  Swz swz;
  int64_t E_D, E_R;
};

// Relayout plan: one loop nest shared by source and destination (their common refinement),
// enumerated fastest digit first.  Addresses in units of `unit_bytes`.
struct RelayoutPlan {
  int32_t n;                       // loop digits decoded from the thread index
  uint32_t ext[kMaxJoint];
  int32_t shift[kMaxJoint];        // log2(ext) when ext is a power of two, else -1
  int64_t ss[kMaxJoint], ds[kMaxJoint];
  int32_t U;                       // per-thread unroll digit (extent U, strides us / ud)
  int64_t us, ud;
  int64_t s_off, d_off;
  Swz s_swz, d_swz;
  int32_t n_r;                     // destination replicas
  int32_t rext[kMaxR];
  int64_t rstr[kMaxR];
  int64_t E_R;
  uint64_t threads;                // total work items = elements / (vector width * U)
  int32_t streaming;               // 1: non-temporal loads and stores (data larger than the caches)
};

// Relayout of rows that are contiguous on both sides and start anywhere: run elements each, the other digits (fastest first) as
// in RelayoutPlan.  A wave takes four slots, a slot 64 16-byte chunks of one row, cut at 16-byte boundaries of the destination.
struct RowPlan {
  int32_t n;
  uint32_t ext[kMaxJoint];
  int64_t ss[kMaxJoint], ds[kMaxJoint];
  int64_t s_off, d_off;
  int64_t run;
  uint32_t slots_per_row, rows;
  uint64_t slots;                  // rows * slots_per_row
};

// Neighbours along the source on one XCD.  Source rows that start anywhere are cut by tiles inside a line (a tile's 128 bytes of a row lie on two), and
// workgroups go round the 8 XCDs one by one, so the two tiles that need such a line used to fetch it into two L2s.  Here runs of 2^run tiles
// fall to one XCD, side by side and at one step of the diagonal: the tile index along the source is permuted inside windows of 8 x 2^run workgroups,
// where there is a window's worth of tiles (TransposePlan::run).  us, one by one -> runs of 4: bf16 5000 x 5001 25.6 -> 23.6, 1959 x 1889 7.2 -> 6.9, bytes 8191 x 8193 38 -> 34,
// 6001 x 4001 14.2 -> 11.6; the skewed kernel, runs of 8: bf16 6001 x 9001 65 -> 51, 8193 x 7999 75 -> 65, 8184 x 8200 61 -> 56, fp32 5001 x 7001 63 -> 59, 8191 x 8193 56
// either way.  Longer runs of the chunk kernel are level or behind (bytes 6001 x 4001 13.9); with 9 tiles along the source 8193 x 1025 is 9.6, and 10.4 when
// the diagonal is made coarser all the same.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline uint32_t tile_in_runs(uint32_t ts, uint32_t n, int run) {
  const uint32_t window = 8u << run;
  return ts < (n & ~(window - 1)) ? (ts & ~(window - 1)) | ((ts & 7) << run) | ((ts >> 3) & ((1u << run) - 1)) : ts;
}

// Transposing relayout: the joint loop nest has one digit that is contiguous in the source (extent
// eS, destination stride dS) and another that is contiguous in the destination (extent eD, source
// stride sD).  A workgroup moves one T x T tile of those two digits through LDS; the other digits
// (fastest first) are decoded from the workgroup index.  Addresses in elements.
struct TransposePlan {
  int32_t n;
  uint32_t ext[kMaxJoint];
  int64_t ss[kMaxJoint], ds[kMaxJoint];
  int64_t eS, eD, sD, dS;
  int64_t s_off, d_off;
  uint32_t tiles_s, tiles_d;       // tiles along the source-fast and the destination-fast digit
  uint32_t grid_s;                 // workgroups along the source: tiles_s, or more of which the last ones only return
  uint64_t blocks;                 // workgroups launched: grid_s * tiles_d * product of ext[]
  int32_t streaming;               // 1: non-temporal loads and stores
  int32_t diag;                    // g > 0: tiles are walked diagonally, td = (row + (ts >> run) / g) mod tiles_d; 0: row by row
  int32_t run;                     // runs of 2^run tiles along S fall to one XCD (tile_in_runs); variants 2 and 3
  Swz s_swz, d_swz;                // swizzle stages of the two sides (mask 0: none), applied to an access's first element
  int32_t n_r;                     // destination replicas: every replica address is written
  int32_t rext[kMaxR];
  int64_t rstr[kMaxR];
  int64_t E_R;
  int32_t elementwise;             // 0: aligned 16-byte chunks; 1: tiles of 64 x 64 moved element by element (any strides, any swizzle);
                                   // 2: 16-byte chunks that start at any element (no swizzle); 3: the same, tiles skewed onto the destination's lines
};

// Fallback when the two digit systems have no common refinement: decode each side separately.
struct GenericRelayoutPlan {
  int32_t ns, nd;
  int64_t sext[kMaxD], sstr[kMaxD];
  int64_t dext[kMaxD], dstr[kMaxD];
  int64_t s_off, d_off;
  Swz s_swz, d_swz;
  int32_t n_r;
  int32_t rext[kMaxR];
  int64_t rstr[kMaxR];
  int64_t E_R;
  int64_t total;
};

// GEMM arguments (addresses in elements of the operand's dtype).
struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  int64_t M, N, K;
  int64_t lda, ldb, ldc;           // row pitch of A (per i), of B's memory image (per j), of C (per i)
  const float* scale_a;            // (ceil(M/128), nkb) or null; bytes (E8M0 codes) when scale_e8m0
  const float* scale_b;            // (ceil(N/128), nkb) or null
  int32_t scale_e8m0;              // 1: the scale arrays hold one E8M0 byte per block (2^(code - 127))
  int32_t scale_a_rows;            // rows of A that share a scale: 128, or 1 (scale_a is then (M, nkb))
  int32_t nkb;
  int32_t out_bf16;                // 0: fp32 output, 1: 16-bit output (bf16, or binary16 when f16 is set)
  int32_t f16;                     // 1: 16-bit inputs (and a 16-bit output) are IEEE binary16 instead of bf16
  int32_t fp8;                     // grouped streaming kernel: 1 = e4m3 inputs (K-tiles of 128 elements), bf16 output
  int32_t grid_m, grid_n;          // workgroup tiles along M and N
  int32_t tile_n;                  // columns of C per workgroup tile (64, 224 or 256)
  // tile family, dense (tile_family.h)
  TileMap map;                     // its map from workgroups to tiles
  int32_t c_vec;                   // 1: C's fragments go out as buffer stores of 4 columns a lane; 0: any N, any pitch
  // 256-tile bf16 kernel: operands pre-tiled along K / blocked along rows (plain matrix: kstep 128, shift 0,
  // blk_stride = tile rows x pitch)
  int32_t a_kstep, b_kstep;        // bytes between consecutive 64-wide K-tiles of one row
  int32_t a_tpb_shift, b_tpb_shift;  // log2(tiles per row block)
  int64_t a_blk_stride, b_blk_stride;  // elements between row blocks
  // grouped GEMM only: group e owns rows group_rows[e] .. group_rows[e + 1] - 1 of A and C and the matrix B + e * ldg
  const int32_t* group_rows;       // device, groups + 1 entries
  int32_t groups;
  int32_t tile_m;                  // rows of a tile of the grouped tile kernel: 128, 256, or 0 = chosen from M / groups
  int32_t compact_groups;          // streaming kernel: blockIdx.y counts non-empty groups (set by its launcher when M < groups)
  int32_t gated;                   // 1: store silu(gate) * up (B's rows interleave gate and up in runs of 16), C is N / 2 wide
  int64_t ldg;
  int32_t stream_b;                // 1: the groups' weights are too many to stay in the last-level cache from one call to the next
  int32_t* clear;                  // streaming kernel, narrow tiles: a word they set to zero (a pair's status), or null
};

// Hand-over between the two grouped GEMMs of a fused pair (the first GEMM's output is the second GEMM's A).  A row
// block of the second GEMM may be read once every column tile of the first GEMM for those rows has been stored:
// done[r] counts the stored column tiles of the row block whose first row is r (both GEMMs cut the groups into row
// blocks of the same height, so the two agree on r); done[M] counts waits that gave up.  Device memory, M + 1
// words, zero when the kernel starts.
struct PairSync {
  int32_t* done;
  int32_t need;                    // column tiles of the first GEMM per row block
  int32_t spin_limit;              // polls of done[r] before a wait gives up (the tile is then computed from what is there)
  int64_t M;
};

}  // namespace axe
