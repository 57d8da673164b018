// Integer kernels: layout evaluation (Def. 2.3) and relayout copies (`copy` operator, Sec. 3.2).
// gfx950 only.  Bandwidth-bound: no LDS, 128-bit global accesses wherever the layouts allow.
#include <hip/hip_runtime.h>

#include "device_types.h"
#include "kernels.h"

namespace axe {

__device__ __forceinline__ int64_t swz_apply(int64_t x, Swz z) {
  return x ^ (((x >> z.shift) & (int64_t)z.mask) << z.base);
}

// ------------------------------------------------------------------------------------------
// Layout evaluation: one thread per logical index.  Digits are peeled from the fastest iter
// (d_i = floor(x / p_i) mod e_i, App. A), each contributes digit * stride to its axis.
// ------------------------------------------------------------------------------------------
template <typename IdxT>
__global__ __launch_bounds__(256) void layout_eval_kernel(EvalDesc d, int64_t n, const int64_t* __restrict__ idx,
                                                          int64_t* __restrict__ out) {
  const int64_t per = d.E_R * d.n_axes;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int64_t x = idx ? idx[i] : i;
    int64_t* o = out + i * per;
    if (x < 0 || x >= d.E_D) {
      for (int64_t t = 0; t < per; ++t) o[t] = INT64_MIN;
      continue;
    }
    int64_t c[kMaxAxes];
#pragma unroll
    for (int a = 0; a < kMaxAxes; ++a) c[a] = d.off[a];
    IdxT rem = (IdxT)x;
    for (int k = d.n_d - 1; k >= 0; --k) {
      IdxT e = (IdxT)d.ext[k];
      IdxT q = rem / e;
      int64_t v = (int64_t)(rem - q * e) * d.str[k];
      rem = q;
      int ax = d.axis[k];
#pragma unroll
      for (int a = 0; a < kMaxAxes; ++a) c[a] += (a == ax) ? v : 0;
    }
    for (int64_t t = 0; t < d.E_R; ++t) {
      int64_t r[kMaxAxes];
#pragma unroll
      for (int a = 0; a < kMaxAxes; ++a) r[a] = c[a];
      int64_t tr = t;
      for (int k = d.n_r - 1; k >= 0; --k) {
        int64_t q = tr / d.rext[k];
        int64_t v = (tr - q * d.rext[k]) * d.rstr[k];
        tr = q;
        int ax = d.raxis[k];
#pragma unroll
        for (int a = 0; a < kMaxAxes; ++a) r[a] += (a == ax) ? v : 0;
      }
#pragma unroll
      for (int a = 0; a < kMaxAxes; ++a) {
        if (a < d.n_axes) {
          int64_t v = r[a];
          if (a == d.swz_axis) v = swz_apply(v, d.swz);
          o[t * d.n_axes + a] = v;
        }
      }
    }
  }
}

// The common case -- no replicas, fewer than 2^31 points, at most 4 axes -- without the generic loop's
// 64-bit divisions and 8-way axis selects: digits in 32 bits (a shift and a mask where the extent is a
// power of two, a multiplication otherwise: 2816 x 5504 points of a tiled layout, 124 MB, 33 us with 32-bit divisions,
// 23 now), one 64-bit multiply-add per digit, the axis loop unrolled to NAX.  A thread evaluates
// PTS consecutive indices (4 when there is a single axis: two 16-byte stores), so that an iter's
// parameters are fetched once for all of them.  Bound: the 8 NAX bytes written per index.
template <int NAX, int PTS>
__global__ __launch_bounds__(256) void layout_eval_fast_kernel(EvalDesc d, int64_t n, const int64_t* __restrict__ idx,
                                                               int64_t* __restrict__ out) {
  // index of the thread's p-th point: a wave owns 64 PTS consecutive indices; with one axis a lane takes pairs
  // (2 lane, 2 lane + 1) 128 apart, so that every store instruction of the wave writes 1 contiguous KiB;
  // otherwise lane-interleaved single indices (each store instruction 64 NAX x 8 contiguous bytes).
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(t & 63);
  const int64_t wbase = (t >> 6) * (64 * PTS);
  auto index_of = [&](int p) -> int64_t {
    return (NAX == 1 && PTS % 2 == 0) ? wbase + (p >> 1) * 128 + lane * 2 + (p & 1) : wbase + p * 64 + lane;
  };
  if (wbase >= n) return;
  int64_t x[PTS], c[PTS][NAX];
  uint32_t rem[PTS];
#pragma unroll
  for (int p = 0; p < PTS; ++p) {
    const int64_t ip = index_of(p);
    const int64_t i = ip < n ? ip : n - 1;                         // (a ragged tail repeats the last index; not stored)
    x[p] = idx ? idx[i] : i;
    rem[p] = (uint32_t)x[p];
#pragma unroll
    for (int a = 0; a < NAX; ++a) c[p][a] = d.off[a];
  }
  // digits outermost: an iter's parameters are fetched once for the thread's PTS indices
  for (int k = d.n_d - 1; k >= 0; --k) {
    const int sh = d.shift[k];
    const uint32_t e = (uint32_t)d.ext[k];
    const int64_t st = d.str[k];
    const int ax = d.axis[k];
    const Div31 by = d.div[k];                                     // (fetched with the others: on demand it is waited for by itself)
#pragma unroll
    for (int p = 0; p < PTS; ++p) {
      uint32_t dig;
      if (sh >= 0) {
        dig = rem[p] & (e - 1u);
        rem[p] >>= sh;
      } else {
        const uint32_t q = div31(rem[p], by);
        dig = rem[p] - q * e;
        rem[p] = q;
      }
      const int64_t v = (int64_t)dig * st;
      if (NAX == 1) {
        c[p][0] += v;
      } else {
#pragma unroll
        for (int a = 0; a < NAX; ++a) c[p][a] += (a == ax) ? v : 0;
      }
    }
  }
#pragma unroll
  for (int p = 0; p < PTS; ++p) {
    const bool bad = x[p] < 0 || x[p] >= d.E_D;
#pragma unroll
    for (int a = 0; a < NAX; ++a) {
      int64_t v = c[p][a];
      if (a == d.swz_axis) v = swz_apply(v, d.swz);
      c[p][a] = bad ? INT64_MIN : v;
    }
  }
  typedef __attribute__((ext_vector_type(2))) int64_t i64x2;
  if (NAX == 1 && PTS % 2 == 0) {                                  // out is 16-byte aligned (the host checks), the pair's first index is even
#pragma unroll
    for (int p = 0; p < PTS; p += 2) {
      const int64_t ip = index_of(p);
      if (ip + 1 < n) __builtin_nontemporal_store(i64x2{c[p][0], c[p + 1][0]}, (i64x2*)(out + ip));
      else if (ip < n) out[ip] = c[p][0];
    }
  } else {
#pragma unroll
    for (int p = 0; p < PTS; ++p) {
      const int64_t ip = index_of(p);
      if (ip < n) {
#pragma unroll
        for (int a = 0; a < NAX; ++a) __builtin_nontemporal_store(c[p][a], &out[ip * NAX + a]);
      }
    }
  }
}

// Replicas, or more axes than the fast kernel takes (fewer than 2^31 points): the per = E_R n_axes words of an index are
// consecutive in the output, so one thread per index would scatter 8-byte stores per x 8 bytes apart.  Here a workgroup
// evaluates D + O of 256 indices once, one per thread (32-bit digits, as above), parks the coordinates in LDS, and writes the
// 256 per words as 16-byte pairs, consecutive lanes on consecutive pairs: a thread keeps its two (replica, axis) positions for
// the whole block -- the stride between its pairs is a multiple of per -- so the replica's offset is worked out once and a word
// costs one LDS read and one addition.  Bound: the 8 per bytes written per index.  2048 x 4096 points of a 4-axis layout with
// two replicas (537 MB): 300 -> 81 us (6.6 TB/s).
template <int NAX>
__global__ __launch_bounds__(256) void layout_eval_block_kernel(EvalDesc d, int64_t n, const int64_t* __restrict__ idx, int64_t* __restrict__ out) {
  typedef __attribute__((ext_vector_type(2))) int64_t i64x2;
  __shared__ int64_t coord[256 * NAX];
  __shared__ uint8_t outside[256];
  const int tid = threadIdx.x;
  const int per = (int)d.E_R * NAX;
  // pairs of words that the workgroup writes at a time: whole indices, an even number of words
  int words = 512 / per * per;
  if (words & 1) words -= per;
  const int step = words / per;                                    // indices between two pairs of a thread
  const bool writes = 2 * tid < words;
  int di[2] = {0, 0}, ax[2] = {0, 0};
  int64_t ro[2] = {0, 0};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = 2 * tid + h;
    di[h] = q / per;
    int t = (q - di[h] * per) / NAX;
    ax[h] = q % NAX;                                               // (per is a multiple of NAX)
    for (int k = d.n_r - 1; k >= 0; --k) {
      const int e = (int)d.rext[k], p = t / e;
      if (d.raxis[k] == ax[h]) ro[h] += (int64_t)(t - p * e) * d.rstr[k];
      t = p;
    }
  }
  for (int64_t b0 = (int64_t)blockIdx.x * 256; b0 < n; b0 += (int64_t)gridDim.x * 256) {
    const int count = n - b0 < 256 ? (int)(n - b0) : 256;
    {
      const int64_t x = tid < count ? (idx ? idx[b0 + tid] : b0 + tid) : 0;
      int64_t c[NAX];
#pragma unroll
      for (int a = 0; a < NAX; ++a) c[a] = d.off[a];
      uint32_t rem = (uint32_t)x;
      for (int k = d.n_d - 1; k >= 0; --k) {
        const uint32_t e = (uint32_t)d.ext[k];
        const Div31 by = d.div[k];
        uint32_t dig;
        if (d.shift[k] >= 0) {
          dig = rem & (e - 1u);
          rem >>= d.shift[k];
        } else {
          const uint32_t q = div31(rem, by);
          dig = rem - q * e;
          rem = q;
        }
        const int64_t v = (int64_t)dig * d.str[k];
#pragma unroll
        for (int a = 0; a < NAX; ++a) c[a] += a == d.axis[k] ? v : 0;
      }
#pragma unroll
      for (int a = 0; a < NAX; ++a) coord[tid * NAX + a] = c[a];
      outside[tid] = x < 0 || x >= d.E_D;
    }
    __syncthreads();
    if (writes) {
      auto word = [&](int i, int h) __attribute__((always_inline)) -> int64_t {
        int64_t v = coord[(i + di[h]) * NAX + ax[h]] + ro[h];
        if (ax[h] == d.swz_axis) v = swz_apply(v, d.swz);
        return outside[i + di[h]] ? INT64_MIN : v;
      };
      int64_t* o = out + b0 * per + 2 * tid;
      for (int i = 0; i < count; i += step, o += words) {
        if (i + di[1] < count) __builtin_nontemporal_store(i64x2{word(i, 0), word(i, 1)}, (i64x2*)o);
        else if (i + di[0] < count) *o = word(i, 0);
      }
    }
    __syncthreads();
  }
}

hipError_t launch_layout_eval(const EvalDesc& d, int64_t n, const int64_t* idx, int64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (d.use32 && d.E_R == 1 && d.n_r == 0 && d.n_axes <= 4 && n < (int64_t(1) << 40)) {
    const bool vec = d.n_axes == 1 && ((uintptr_t)out & 15) == 0;  // 4 indices per thread, two 16-byte stores
    const int pts = d.n_axes == 1 ? (vec ? 4 : 1) : 2;
    const int64_t threads = (n + pts - 1) / pts;
    const dim3 grid((unsigned)((threads + 255) / 256)), block(256);
    switch (d.n_axes * 2 + (vec ? 1 : 0)) {
      case 3: hipLaunchKernelGGL((layout_eval_fast_kernel<1, 4>), grid, block, 0, s, d, n, idx, out); break;
      case 2: hipLaunchKernelGGL((layout_eval_fast_kernel<1, 1>), grid, block, 0, s, d, n, idx, out); break;
      case 4: hipLaunchKernelGGL((layout_eval_fast_kernel<2, 2>), grid, block, 0, s, d, n, idx, out); break;
      case 6: hipLaunchKernelGGL((layout_eval_fast_kernel<3, 2>), grid, block, 0, s, d, n, idx, out); break;
      default: hipLaunchKernelGGL((layout_eval_fast_kernel<4, 2>), grid, block, 0, s, d, n, idx, out); break;
    }
    return hipGetLastError();
  }
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536 * 4) blocks = 65536 * 4;
  if (layout_eval_by_blocks(d, n, out)) {
    const dim3 grid((unsigned)blocks), block(256);
    switch (d.n_axes) {
      case 1: hipLaunchKernelGGL(layout_eval_block_kernel<1>, grid, block, 0, s, d, n, idx, out); break;
      case 2: hipLaunchKernelGGL(layout_eval_block_kernel<2>, grid, block, 0, s, d, n, idx, out); break;
      case 3: hipLaunchKernelGGL(layout_eval_block_kernel<3>, grid, block, 0, s, d, n, idx, out); break;
      case 4: hipLaunchKernelGGL(layout_eval_block_kernel<4>, grid, block, 0, s, d, n, idx, out); break;
      case 5: hipLaunchKernelGGL(layout_eval_block_kernel<5>, grid, block, 0, s, d, n, idx, out); break;
      case 6: hipLaunchKernelGGL(layout_eval_block_kernel<6>, grid, block, 0, s, d, n, idx, out); break;
      case 7: hipLaunchKernelGGL(layout_eval_block_kernel<7>, grid, block, 0, s, d, n, idx, out); break;
      default: hipLaunchKernelGGL(layout_eval_block_kernel<8>, grid, block, 0, s, d, n, idx, out); break;
    }
    return hipGetLastError();
  }
  if (d.use32)
    hipLaunchKernelGGL(layout_eval_kernel<uint32_t>, dim3((unsigned)blocks), dim3(256), 0, s, d, n, idx, out);
  else
    hipLaunchKernelGGL(layout_eval_kernel<uint64_t>, dim3((unsigned)blocks), dim3(256), 0, s, d, n, idx, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Relayout, joint loop nest.  Thread w decodes its digits (fastest first); its U unrolled
// elements step along one more digit.  All loads are issued before the first store.
// ------------------------------------------------------------------------------------------
template <int BYTES> struct Word;
template <> struct Word<1> { using T = uint8_t; };
template <> struct Word<2> { using T = uint16_t; };
template <> struct Word<4> { using T = uint32_t; };
template <> struct Word<8> { using T = __attribute__((ext_vector_type(2))) uint32_t; };
template <> struct Word<16> { using T = __attribute__((ext_vector_type(4))) uint32_t; };

template <int EB>
struct Row {                                                       // a 16-byte chunk as elements
  typename Word<EB>::T w[16 / EB];
};

template <int BYTES, int U, bool REPL, bool NT>
__global__ __launch_bounds__(256) void relayout_joint_kernel(RelayoutPlan p, const void* __restrict__ src_,
                                                             void* __restrict__ dst_) {
  using T = typename Word<BYTES>::T;
  const T* __restrict__ src = (const T*)src_;
  T* __restrict__ dst = (T*)dst_;
  uint64_t w64 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w64 >= p.threads) return;
  uint32_t w = (uint32_t)w64;            // host guarantees threads < 2^32
  int64_t s = p.s_off, d = p.d_off;
  for (int k = 0; k < p.n; ++k) {
    uint32_t dig;
    if (p.shift[k] >= 0) {
      dig = w & (p.ext[k] - 1);
      w >>= p.shift[k];
    } else {
      uint32_t q = w / p.ext[k];
      dig = w - q * p.ext[k];
      w = q;
    }
    s += (int64_t)dig * p.ss[k];
    d += (int64_t)dig * p.ds[k];
  }
  T v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const T* a = &src[swz_apply(s + u * p.us, p.s_swz)];
    v[u] = NT ? __builtin_nontemporal_load(a) : *a;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    int64_t da = d + u * p.ud;
    if (!REPL) {
      T* a = &dst[swz_apply(da, p.d_swz)];
      if (NT) __builtin_nontemporal_store(v[u], a);
      else *a = v[u];
    } else {
      for (int64_t t = 0; t < p.E_R; ++t) {
        int64_t tr = t, ra = da;
        for (int k = p.n_r - 1; k >= 0; --k) {
          int64_t q = tr / p.rext[k];
          ra += (tr - q * p.rext[k]) * p.rstr[k];
          tr = q;
        }
        dst[swz_apply(ra, p.d_swz)] = v[u];
      }
    }
  }
}

template <int BYTES, int U>
static hipError_t launch_joint_u(const RelayoutPlan& p, const void* src, void* dst, hipStream_t s) {
  unsigned blocks = (unsigned)((p.threads + 255) / 256);
  if (p.n_r > 0)
    hipLaunchKernelGGL((relayout_joint_kernel<BYTES, U, true, false>), dim3(blocks), dim3(256), 0, s, p, src, dst);
  else if (p.streaming)
    hipLaunchKernelGGL((relayout_joint_kernel<BYTES, U, false, true>), dim3(blocks), dim3(256), 0, s, p, src, dst);
  else
    hipLaunchKernelGGL((relayout_joint_kernel<BYTES, U, false, false>), dim3(blocks), dim3(256), 0, s, p, src, dst);
  return hipGetLastError();
}

template <int BYTES>
static hipError_t launch_joint_b(const RelayoutPlan& p, const void* src, void* dst, hipStream_t s) {
  switch (p.U) {
    case 1: return launch_joint_u<BYTES, 1>(p, src, dst, s);
    case 2: return launch_joint_u<BYTES, 2>(p, src, dst, s);
    case 4: return launch_joint_u<BYTES, 4>(p, src, dst, s);
    case 8: return launch_joint_u<BYTES, 8>(p, src, dst, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_relayout_joint(const RelayoutPlan& p, int unit_bytes, const void* src, void* dst, hipStream_t s) {
  if (p.threads == 0) return hipSuccess;
  switch (unit_bytes) {
    case 1: return launch_joint_b<1>(p, src, dst, s);
    case 2: return launch_joint_b<2>(p, src, dst, s);
    case 4: return launch_joint_b<4>(p, src, dst, s);
    case 8: return launch_joint_b<8>(p, src, dst, s);
    case 16: return launch_joint_b<16>(p, src, dst, s);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------------------------------
// Relayout of contiguous rows whose length, pitch or start is no multiple of 16 bytes (padding an odd matrix, cutting a
// window out of one).  The loop nest above moves such rows in the largest unit that divides everything, single elements at
// worst.  Here a lane moves a 16-byte chunk of the destination, aligned there, loaded from wherever it starts in the
// source (global memory takes any address); the chunk a row begins or ends in is loaded from inside the row, shifted,
// and stored element by element.  Which row a wave is at is worked out once for four slots of 64 chunks, on uniform
// values: the divisions would otherwise be most of the work.  Bound: HBM.  us, rotating over three pairs of buffers: bf16
// 8191 x 8191 to rows on whole lines 190 -> 51 (5.3 TB/s), bytes 8191 x 8190 99 -> 28, fp32 4097 x 4095 58 -> 28, 8-byte 62 -> 53,
// bf16 4450 x 943 8.5 -> 6.3.
// ------------------------------------------------------------------------------------------
template <int EB>
__global__ __launch_bounds__(256) void relayout_rows_kernel(RowPlan p, const uint8_t* __restrict__ src, uint8_t* __restrict__ dst) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  typedef u32x4 u32x4_any __attribute__((aligned(1)));
  using W = typename Word<EB>::T;
  constexpr int CE = 16 / EB, U = kRowSlots / 4;                   // slots of a wave
  const int lane = threadIdx.x & 63;
  const uint64_t t = ((uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * U;
  if (t >= p.slots) return;
  uint32_t row = (uint32_t)(t / p.slots_per_row), seg = (uint32_t)(t - (uint64_t)row * p.slots_per_row);
  const int64_t bytes = p.run * EB;
  const uint8_t* s = nullptr;
  uint8_t* d = nullptr;
  auto locate = [&]() __attribute__((always_inline)) {            // start of the row on either side
    int64_t so = p.s_off, dof = p.d_off;
    uint32_t rem = row;
    for (int k = 0; k < p.n; ++k) {
      const uint32_t q = rem / p.ext[k], dig = rem - q * p.ext[k];
      so += (int64_t)dig * p.ss[k];
      dof += (int64_t)dig * p.ds[k];
      rem = q;
    }
    s = src + so * EB, d = dst + dof * EB;
  };
  locate();
  u32x4 held[U];
  uint8_t* at[U];
  int64_t off[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    at[u] = d;
    off[u] = bytes;                                                // (no such slot: nothing to store)
    if (row < p.rows) {
      const int64_t o = ((int64_t)seg * 64 + lane) * 16 - ((uintptr_t)d & 15);   // byte of the row the chunk begins at
      const int64_t in = o < 0 ? 0 : (o + 16 <= bytes ? o : bytes - 16);         // the nearest chunk inside the row
      held[u] = *(const u32x4_any*)(s + in);
      off[u] = o;
      if (++seg == p.slots_per_row) {
        seg = 0, ++row;
        if (u + 1 < U && row < p.rows) locate();
      }
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t o = off[u];
    if (o >= bytes) continue;
    if (o >= 0 && o + 16 <= bytes) {
      *(u32x4*)(at[u] + o) = held[u];
    } else {
      unsigned __int128 x = __builtin_bit_cast(unsigned __int128, held[u]);
      x = o < 0 ? x << (int)(-o * 8) : x >> (int)((o + 16 - bytes) * 8);
      const Row<EB> e = __builtin_bit_cast(Row<EB>, x);
#pragma unroll
      for (int k = 0; k < CE; ++k)
        if (o + k * EB >= 0 && o + k * EB < bytes) *(W*)(at[u] + o + k * EB) = e.w[k];
    }
  }
}

hipError_t launch_relayout_rows(const RowPlan& p, int elem_bytes, const void* src, void* dst, hipStream_t s) {
  if (p.slots == 0) return hipSuccess;
  const uint64_t blocks = (p.slots + kRowSlots - 1) / kRowSlots;
  if (blocks > kMaxBlocks256) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  const uint8_t* from = (const uint8_t*)src;
  uint8_t* to = (uint8_t*)dst;
  switch (elem_bytes) {
    case 1: hipLaunchKernelGGL(relayout_rows_kernel<1>, grid, block, 0, s, p, from, to); break;
    case 2: hipLaunchKernelGGL(relayout_rows_kernel<2>, grid, block, 0, s, p, from, to); break;
    case 4: hipLaunchKernelGGL(relayout_rows_kernel<4>, grid, block, 0, s, p, from, to); break;
    case 8: hipLaunchKernelGGL(relayout_rows_kernel<8>, grid, block, 0, s, p, from, to); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Relayout, transposing: source and destination are contiguous along different digits of the joint
// loop nest (row-major <-> column-major and their batched, strided relatives).  Moving single
// elements would leave one side with 2-byte accesses scattered over rows; instead a workgroup
// takes a T x T tile of the two digits, reads it with 16-byte loads along the source-fast digit
// (T * EB = 128 to 512 contiguous bytes per tile row), parks it in LDS, and writes it with 16-byte
// stores along the destination-fast digit, each store gathering its 16 / EB elements from as many
// LDS rows.  The LDS image is XOR-swizzled, not padded: 16-byte chunk c of row r sits at chunk position
// c ^ (r / elements per chunk), which keeps the gather on distinct banks for every element size.
// ------------------------------------------------------------------------------------------
//
// ANY: the same tiles where extents, strides, offsets or buffers are no multiples of a chunk (odd matrix sizes): the 16-byte
// accesses start at any element (global memory takes them), a chunk that sticks out of the tensor is loaded from the last
// place inside it and shifted, and stored element by element.  The rows of neighbouring tiles then share lines of the
// destination: ordinary stores (non-temporal ones do not combine), and the grid may be padded to whole rounds of the 8 XCDs
// along the source (grid_s), so that the tiles that complete a line meet in one XCD's L2.  us, element by element -> now, rotating over
// three pairs of buffers: bf16 7000 x 3001 27 -> 19 (4.4 TB/s), 4095 x 4097 20.6 -> 15.5, bytes 8191 x 8193 70 -> 40, bf16 105 -> 83 (a band of
// tiles along the destination per XCD instead of the padding: 93).
template <int EB, bool NT, bool ANY>
__global__ __launch_bounds__(256) void relayout_transpose_kernel(TransposePlan p, const uint8_t* __restrict__ src,
                                                                 uint8_t* __restrict__ dst) {
  constexpr int T = EB == 8 ? 64 : 128;                           // tile edge, elements (transpose_tile_edge)
  constexpr int CE = 16 / EB;                                    // elements per 16-byte chunk
  constexpr int CPR = T / CE;                                    // chunks per tile row
  constexpr int ROWB = T * EB;                                   // bytes of a tile row in LDS
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  typedef u32x4 u32x4_any __attribute__((aligned(1)));
  // LDS image of the tile: rows of ROWB bytes, the 16-byte chunk c of row r at chunk position c ^ (r / CE) -- the
  // same kind of XOR stage as the swizzled layouts of the GEMM tiles.  Rows come in whole chunks (one 16-byte
  // write each); on the way out a lane gathers the CE elements of its chunk from CE consecutive rows at one
  // column, and the 16 (or more) lanes that do so for neighbouring chunks sit CE rows apart: their keys differ,
  // so they read different banks (a padded pitch cannot do that for 1- and 2-byte elements: CE x pitch is a
  // multiple of 8 words, and two of every 16 lanes met in a bank).  Measured: the conflict counter drops to
  // zero.
  __shared__ __attribute__((aligned(16))) uint8_t tile[T * ROWB];
  auto lds_at = [&](int row, int byte_col, int key) -> uint8_t* {
    return tile + row * ROWB + ((((byte_col >> 4) ^ key) & (CPR - 1)) << 4) + (byte_col & 15);
  };

  // workgroup -> (tile along S, tile along D, outer digits)
  uint64_t b = blockIdx.x;
  uint32_t ts = (uint32_t)(b % p.grid_s);
  if (ANY && p.run) ts = tile_in_runs(ts, p.grid_s, p.run);
  if (ANY && ts >= p.tiles_s) return;
  b /= p.grid_s;
  uint32_t td = (uint32_t)(b % p.tiles_d);
  b /= p.tiles_d;
  // Row by row (ts fastest, td fixed for tiles_s workgroups in a row) the workgroups running at one time read
  // whole rows of the source between them, but write one narrow column of the destination: short segments a row
  // pitch apart, which with power-of-two pitches fall on a fraction of the memory channels.  Walking the tiles
  // diagonally gives every window of workgroups many different td as well as many different ts.
  // (p.run is 0 where chunks are aligned.  Reading it costs fp32 there a wait before the first load: 292 x 48 4.40 us -> 4.62, bytes and
  // 8-byte elements 1 %; the 2-byte kernel's code comes out 1 - 1.5 % faster with it, 512 x 512 4.23 -> 4.16.)
  if (p.diag > 0) td = (td + (ANY || EB == 2 ? ts >> p.run : ts) / (uint32_t)p.diag) % p.tiles_d;
  int64_t sb = p.s_off, db = p.d_off;
  for (int k = 0; k < p.n; ++k) {
    const uint64_t q = b / p.ext[k];
    const int64_t dig = (int64_t)(b - q * p.ext[k]);
    sb += dig * p.ss[k];
    db += dig * p.ds[k];
    b = q;
  }
  const int64_t s0 = (int64_t)ts * T, d0 = (int64_t)td * T;      // tile origin in the two digits

  // HBM -> LDS: row r of the tile is destination-fast index d0 + r, its chunks run along the source.  All loads
  // of a thread are issued before the first of them is waited for: with one load at a time in flight per thread
  // the kernel was bound by the latency of HBM (4.1 - 4.2 TB/s on 8192 x 8192 bf16, whatever the LDS layout or the
  // order of the tiles), not by its bandwidth.
  constexpr int NL = T * CPR / 256;                              // chunks per thread
  u32x4 held[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int c = (int)threadIdx.x + 256 * i;
    const int r = c / CPR, cc = c % CPR;
    const int64_t iD = d0 + r, iS = s0 + (int64_t)cc * CE;
    // extents are multiples of CE: a chunk is in or out as a whole.  A chunk outside the tensor is replaced by the
    // tile's first one (always inside) instead of being skipped: a load under a branch would be waited for at
    // the end of that branch, one by one.
    if constexpr (ANY) {                                           // the nearest chunk that lies inside the tensor as a whole
      const int64_t jD = iD < p.eD ? iD : p.eD - 1, jS = iS + CE <= p.eS ? iS : p.eS - CE;
      held[i] = *(const u32x4_any*)(src + (sb + jD * p.sD + jS) * EB);
      continue;
    }
    const bool in = iD < p.eD && iS < p.eS;
    // (a swizzle stage moves whole chunks: the host admits it here only when it leaves the bits inside a chunk alone)
    const u32x4* a = (const u32x4*)(src + swz_apply(sb + (in ? iD * p.sD + iS : d0 * p.sD + s0), p.s_swz) * EB);
    held[i] = NT ? __builtin_nontemporal_load(a) : *a;
  }
  if (ANY && s0 + T > p.eS) {                                      // the last tile along the source: chunks that were moved back
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int64_t over = s0 + (int64_t)((threadIdx.x + 256 * i) % CPR) * CE + CE - p.eS;
      if (over > 0 && over < CE)
        held[i] = __builtin_bit_cast(u32x4, __builtin_bit_cast(unsigned __int128, held[i]) >> (int)(over * EB * 8));
    }
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int c = (int)threadIdx.x + 256 * i;
    const int r = c / CPR, cc = c % CPR;
    *(u32x4*)lds_at(r, cc * 16, r / CE) = held[i];               // (chunks outside the tensor: values nobody reads)
  }
  __syncthreads();
  // LDS -> HBM: output row r is source-fast index s0 + r, its chunks run along the destination
  for (int c = threadIdx.x; c < T * CPR; c += 256) {
    const int r = c / CPR, cc = c % CPR;
    const int64_t iS = s0 + r, iD = d0 + (int64_t)cc * CE;
    if (iS < p.eS && iD < p.eD) {
      // element k of the chunk: LDS row cc * CE + k (key cc), column r
      u32x4 v;
      if (EB == 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          uint32_t w = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) w |= (uint32_t)*lds_at(cc * CE + 4 * j + k, r, cc) << (8 * k);
          v[j] = w;
        }
      } else if (EB == 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t lo = *(const uint16_t*)lds_at(cc * CE + 2 * j, r * 2, cc);
          const uint32_t hi = *(const uint16_t*)lds_at(cc * CE + 2 * j + 1, r * 2, cc);
          v[j] = lo | (hi << 16);
        }
      } else if (EB == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *(const uint32_t*)lds_at(cc * CE + j, r * 4, cc);
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint32_t* q = (const uint32_t*)lds_at(cc * CE + j, r * 8, cc);
          v[2 * j] = q[0];
          v[2 * j + 1] = q[1];
        }
      }
      for (int64_t t = 0; t < p.E_R; ++t) {                        // every replica of the destination (usually one)
        int64_t tr = t, ra = db + iS * p.dS + iD;
        for (int k = p.n_r - 1; k >= 0; --k) {
          ra += (tr % p.rext[k]) * p.rstr[k];
          tr /= p.rext[k];
        }
        if constexpr (ANY) {
          using W = typename Word<EB>::T;
          if (iD + CE <= p.eD) {
            *(u32x4_any*)(dst + ra * EB) = v;
          } else {
#pragma unroll
            for (int k = 0; k < CE; ++k)
              if (iD + k < p.eD) ((W*)dst)[ra + k] = __builtin_bit_cast(Row<EB>, v).w[k];
          }
          continue;
        }
        u32x4* a = (u32x4*)(dst + swz_apply(ra, p.d_swz) * EB);
        if (NT) __builtin_nontemporal_store(v, a);
        else *a = v;
      }
    }
  }
}

// SKEW: destination rows that do not start on 128-byte lines (odd or merely 16-byte aligned pitches).  A tile that ends at the
// same index in every row then ends inside a line in most of them, and a line that two workgroups write in parts costs HBM far
// more than a whole one: 8184 x 8200 bf16, all of whose chunks are aligned, takes 85 us where 8192 x 8192 takes 51.  Here
// every row of the destination has its own boundaries, on lines: the tile of destination index d0 writes [d0 - delta, d0 + TD -
// delta) of a row whose phase in its line is delta, and reads the H = 128 / EB source rows before d0 besides its own TD.  So
// each line is written whole, by eight lanes of one store instruction; the H rows are read twice (mostly from the last-level
// cache).  us, rotating over three pairs: bf16 8191 x 8193 105 (element by element) -> 56 (4.8 TB/s), 8184 x 8200 85 (aligned
// chunks) -> 60, fp32 4095 x 4097 42 -> 30, 8-byte 4095 x 4097 73 -> 51 (5.3 TB/s).
template <int EB, bool NT>
__global__ __launch_bounds__(256) void relayout_transpose_skew_kernel(TransposePlan p, const uint8_t* __restrict__ src, uint8_t* __restrict__ dst) {
  constexpr int TS = skew_tile_s(EB), TD = skew_tile_d(EB);        // elements along the source and along the destination
  constexpr int CE = 16 / EB, H = 128 / EB;                        // elements per chunk, per line
  constexpr int CS = TS / CE, CD = TD / CE;                        // chunks of a tile row on either side
  constexpr int ROWB = TS * EB;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  typedef u32x4 u32x4_any __attribute__((aligned(1)));
  using W = typename Word<EB>::T;
  __shared__ __attribute__((aligned(16))) uint8_t tile[(TD + H) * ROWB];
  // (the image of the kernel above: chunk c of row r at chunk position c ^ (r / CE))
  auto lds_at = [&](int row, int byte_col) -> uint8_t* {
    return tile + row * ROWB + ((((byte_col >> 4) ^ (row / CE)) & (CS - 1)) << 4) + (byte_col & 15);
  };
  uint64_t b = blockIdx.x;
  uint32_t ts = (uint32_t)(b % p.tiles_s);
  if (p.run) ts = tile_in_runs(ts, p.tiles_s, p.run);
  b /= p.tiles_s;
  uint32_t td = (uint32_t)(b % p.tiles_d);
  b /= p.tiles_d;
  if (p.diag > 0) td = (td + (ts >> p.run) / (uint32_t)p.diag) % p.tiles_d;
  int64_t sb = p.s_off, db = p.d_off;
  for (int k = 0; k < p.n; ++k) {
    const uint64_t q = b / p.ext[k];
    const int64_t dig = (int64_t)(b - q * p.ext[k]);
    sb += dig * p.ss[k];
    db += dig * p.ds[k];
    b = q;
  }
  const int64_t s0 = (int64_t)ts * TS, d0 = (int64_t)td * TD;

  // HBM -> LDS: LDS row r is destination-fast index d0 - H + r
  constexpr int NL = (TD + H) * CS / 256;
  static_assert((TD + H) * CS % 256 == 0, "whole trips");
  u32x4 held[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int c = (int)threadIdx.x + 256 * i;
    const int64_t iD = d0 - H + c / CS, iS = s0 + (c % CS) * CE;
    const int64_t jD = iD < 0 ? 0 : (iD < p.eD ? iD : p.eD - 1), jS = iS + CE <= p.eS ? iS : p.eS - CE;   // the nearest place inside the tensor
    held[i] = *(const u32x4_any*)(src + (sb + jD * p.sD + jS) * EB);
  }
  if (s0 + TS > p.eS) {                                            // the last tile along the source: chunks that were moved back
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int64_t over = s0 + (int64_t)((threadIdx.x + 256 * i) % CS) * CE + CE - p.eS;
      if (over > 0 && over < CE)
        held[i] = __builtin_bit_cast(u32x4, __builtin_bit_cast(unsigned __int128, held[i]) >> (int)(over * EB * 8));
    }
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int c = (int)threadIdx.x + 256 * i;
    *(u32x4*)lds_at(c / CS, (c % CS) * 16) = held[i];
  }
  __syncthreads();
  // LDS -> HBM: output row r is source-fast index s0 + r
  for (int c = threadIdx.x; c < TS * CD; c += 256) {
    const int r = c / CD, cc = c % CD;
    const int64_t iS = s0 + r;
    if (iS >= p.eS) continue;
    uint8_t* row = dst + (db + iS * p.dS) * EB;                    // destination index 0 of this row
    const int delta = (int)((uintptr_t)row & 127) / EB;
    const int64_t iD = d0 + cc * CE - delta;
    if (iD + CE <= 0 || iD >= p.eD) continue;
    const int l0 = H + cc * CE - delta;                            // LDS row of the chunk's first element
    W w[CE];
#pragma unroll
    for (int k = 0; k < CE; ++k) w[k] = *(const W*)lds_at(l0 + k, r * EB);
    for (int64_t t = 0; t < p.E_R; ++t) {                          // (replicas lie whole lines apart)
      int64_t tr = t, ro = 0;
      for (int k = p.n_r - 1; k >= 0; --k) {
        ro += (tr % p.rext[k]) * p.rstr[k];
        tr /= p.rext[k];
      }
      uint8_t* at = row + (ro + iD) * EB;
      if (iD >= 0 && iD + CE <= p.eD) {
        const u32x4 v = __builtin_bit_cast(u32x4, w);
        if (NT) __builtin_nontemporal_store(v, (u32x4*)at);
        else *(u32x4*)at = v;
      } else {
#pragma unroll
        for (int k = 0; k < CE; ++k)
          if (iD + k >= 0 && iD + k < p.eD) ((W*)at)[k] = w[k];
      }
    }
  }
}

// The same transposition element by element, for pairs of layouts the 16-byte variant cannot take: extents, strides
// or offsets that are no multiples of a chunk, buffers that are not 16-byte aligned, a swizzle that reaches into a
// chunk.  A workgroup moves a 64 x 64 tile: each wave instruction reads 64 consecutive elements along the
// source-fast digit and writes 64 consecutive elements along the destination-fast digit (the per-element kernel
// leaves one side with single elements scattered over rows); the tile is parked in LDS with a pitch of 65 words.
template <int EB>
__global__ __launch_bounds__(256) void relayout_transpose_elem_kernel(TransposePlan p, const void* __restrict__ src_,
                                                                      void* __restrict__ dst_) {
  constexpr int T = 64;
  using W = typename Word<EB>::T;
  const W* __restrict__ src = (const W*)src_;
  W* __restrict__ dst = (W*)dst_;
  __shared__ W tile[T][T + 1];
  uint64_t b = blockIdx.x;
  const uint32_t ts = (uint32_t)(b % p.tiles_s);
  b /= p.tiles_s;
  uint32_t td = (uint32_t)(b % p.tiles_d);
  b /= p.tiles_d;
  if (p.diag > 0) td = (td + ts / (uint32_t)p.diag) % p.tiles_d;
  int64_t sb = p.s_off, db = p.d_off;
  for (int k = 0; k < p.n; ++k) {
    const uint64_t q = b / p.ext[k];
    const int64_t dig = (int64_t)(b - q * p.ext[k]);
    sb += dig * p.ss[k];
    db += dig * p.ds[k];
    b = q;
  }
  const int64_t s0 = (int64_t)ts * T, d0 = (int64_t)td * T;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  // tile row r: destination-fast index d0 + r, lanes along the source.  All 16 loads of a thread are issued before
  // the first is used (an element outside the tensor is replaced by the tile's first one, always inside: a load
  // under a branch would be waited for at the end of that branch, one by one)
  W held[T / 4];
#pragma unroll
  for (int k = 0; k < T / 4; ++k) {
    const int64_t iD = d0 + ty + 4 * k, iS = s0 + tx;
    const bool in = iD < p.eD && iS < p.eS;
    held[k] = src[swz_apply(sb + (in ? iD * p.sD + iS : d0 * p.sD + s0), p.s_swz)];
  }
#pragma unroll
  for (int k = 0; k < T / 4; ++k) tile[ty + 4 * k][tx] = held[k];
  __syncthreads();
  for (int r = ty; r < T; r += 4) {                              // output row r: source-fast index s0 + r, lanes along the destination
    const int64_t iS = s0 + r, iD = d0 + tx;
    if (iS < p.eS && iD < p.eD) {
      const W v = tile[tx][r];
      for (int64_t t = 0; t < p.E_R; ++t) {
        int64_t tr = t, ra = db + iS * p.dS + iD;
        for (int k = p.n_r - 1; k >= 0; --k) {
          ra += (tr % p.rext[k]) * p.rstr[k];
          tr /= p.rext[k];
        }
        dst[swz_apply(ra, p.d_swz)] = v;               // (ordinary stores: single elements written non-temporally do not combine -- 3.8 -> 1.7 TB/s on bf16)
      }
    }
  }
}

template <int EB>
static hipError_t launch_transpose_e(const TransposePlan& p, const void* src, void* dst, hipStream_t s) {
  if (p.elementwise) {
    hipLaunchKernelGGL((relayout_transpose_kernel<EB, false, true>), dim3((unsigned)p.blocks), dim3(256), 0, s, p, (const uint8_t*)src,
                       (uint8_t*)dst);
  } else if (p.streaming)
    hipLaunchKernelGGL((relayout_transpose_kernel<EB, true, false>), dim3((unsigned)p.blocks), dim3(256), 0, s, p, (const uint8_t*)src,
                       (uint8_t*)dst);
  else
    hipLaunchKernelGGL((relayout_transpose_kernel<EB, false, false>), dim3((unsigned)p.blocks), dim3(256), 0, s, p, (const uint8_t*)src,
                       (uint8_t*)dst);
  return hipGetLastError();
}

hipError_t launch_relayout_transpose(const TransposePlan& p, int elem_bytes, const void* src, void* dst, hipStream_t s) {
  if (p.blocks == 0) return hipSuccess;
  if (p.blocks > kMaxBlocks256) return hipErrorInvalidValue;
  if (p.elementwise == 3) {
    const dim3 grid((unsigned)p.blocks), block(256);
    const uint8_t* from = (const uint8_t*)src;
    uint8_t* to = (uint8_t*)dst;
    switch (elem_bytes * 2 + (p.streaming ? 1 : 0)) {
      case 4: hipLaunchKernelGGL((relayout_transpose_skew_kernel<2, false>), grid, block, 0, s, p, from, to); break;
      case 5: hipLaunchKernelGGL((relayout_transpose_skew_kernel<2, true>), grid, block, 0, s, p, from, to); break;
      case 8: hipLaunchKernelGGL((relayout_transpose_skew_kernel<4, false>), grid, block, 0, s, p, from, to); break;
      case 9: hipLaunchKernelGGL((relayout_transpose_skew_kernel<4, true>), grid, block, 0, s, p, from, to); break;
      case 16: hipLaunchKernelGGL((relayout_transpose_skew_kernel<8, false>), grid, block, 0, s, p, from, to); break;
      case 17: hipLaunchKernelGGL((relayout_transpose_skew_kernel<8, true>), grid, block, 0, s, p, from, to); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  if (p.elementwise == 1) {
    const dim3 grid((unsigned)p.blocks), block(256);
    switch (elem_bytes) {
      case 1: hipLaunchKernelGGL(relayout_transpose_elem_kernel<1>, grid, block, 0, s, p, src, dst); break;
      case 2: hipLaunchKernelGGL(relayout_transpose_elem_kernel<2>, grid, block, 0, s, p, src, dst); break;
      case 4: hipLaunchKernelGGL(relayout_transpose_elem_kernel<4>, grid, block, 0, s, p, src, dst); break;
      case 8: hipLaunchKernelGGL(relayout_transpose_elem_kernel<8>, grid, block, 0, s, p, src, dst); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (elem_bytes) {
    case 1: return launch_transpose_e<1>(p, src, dst, s);
    case 2: return launch_transpose_e<2>(p, src, dst, s);
    case 4: return launch_transpose_e<4>(p, src, dst, s);
    case 8: return launch_transpose_e<8>(p, src, dst, s);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------------------------------
// Relayout, generic: one element per thread, source and destination decoded separately from
// the logical index.  Correct for any pair of layouts; used when no joint loop nest exists.
// ------------------------------------------------------------------------------------------
template <int BYTES>
__global__ __launch_bounds__(256) void relayout_generic_kernel(GenericRelayoutPlan p, const void* __restrict__ src_,
                                                               void* __restrict__ dst_) {
  using T = typename Word<BYTES>::T;
  const T* __restrict__ src = (const T*)src_;
  T* __restrict__ dst = (T*)dst_;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < p.total; x += (int64_t)gridDim.x * blockDim.x) {
    int64_t s = p.s_off, d = p.d_off;
    uint64_t rem = (uint64_t)x;
    for (int k = p.ns - 1; k >= 0; --k) {
      uint64_t q = rem / (uint64_t)p.sext[k];
      s += (int64_t)(rem - q * (uint64_t)p.sext[k]) * p.sstr[k];
      rem = q;
    }
    rem = (uint64_t)x;
    for (int k = p.nd - 1; k >= 0; --k) {
      uint64_t q = rem / (uint64_t)p.dext[k];
      d += (int64_t)(rem - q * (uint64_t)p.dext[k]) * p.dstr[k];
      rem = q;
    }
    T v = src[swz_apply(s, p.s_swz)];
    for (int64_t t = 0; t < p.E_R; ++t) {
      int64_t tr = t, ra = d;
      for (int k = p.n_r - 1; k >= 0; --k) {
        int64_t q = tr / p.rext[k];
        ra += (tr - q * p.rext[k]) * p.rstr[k];
        tr = q;
      }
      dst[swz_apply(ra, p.d_swz)] = v;
    }
  }
}

hipError_t launch_relayout_generic(const GenericRelayoutPlan& p, int unit_bytes, const void* src, void* dst,
                                   hipStream_t s) {
  if (p.total <= 0) return hipSuccess;
  int64_t blocks = (p.total + 255) / 256;
  if (blocks > 65536 * 4) blocks = 65536 * 4;
  dim3 g((unsigned)blocks), b(256);
  switch (unit_bytes) {
    case 1: hipLaunchKernelGGL(relayout_generic_kernel<1>, g, b, 0, s, p, src, dst); break;
    case 2: hipLaunchKernelGGL(relayout_generic_kernel<2>, g, b, 0, s, p, src, dst); break;
    case 4: hipLaunchKernelGGL(relayout_generic_kernel<4>, g, b, 0, s, p, src, dst); break;
    case 8: hipLaunchKernelGGL(relayout_generic_kernel<8>, g, b, 0, s, p, src, dst); break;
    case 16: hipLaunchKernelGGL(relayout_generic_kernel<16>, g, b, 0, s, p, src, dst); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace axe
