// CSR aggregation Y = Abar X (+ Add) (ReLU), the sparse half of eq. (2).
//
// One row of Abar is handled by a group of LPR lanes of a wave (LPR = 64 for
// wide features, fewer for narrow ones, so a wave covers 64 / LPR rows);
// each lane owns VEC consecutive feature columns and walks the row's
// nonzeros, so every nonzero costs one coalesced gather of LPR * VEC floats
// of X.  The row's (col, val) pairs are read cooperatively, one per lane, and
// broadcast within the lane group, so each nonzero's index is loaded once
// per group instead of once per lane.  Features wider than 64 * VEC are split
// into column tiles.  Blocks are ordered XCD-major, column tile major: each
// XCD's L2 sees a contiguous range of rows of one column slab at a time
// (block-ordered graphs keep neighbours close).
// No atomics: every output element is written by exactly one lane.  A row of
// up to kLongRow nonzeros is summed in storage order, a longer one in kSegs
// parts, each in storage order, added in order.  The order is a function of
// the row's length alone: not of the widths, alignments or entry counts that
// choose a kernel, so results are bitwise reproducible across all of them.

#include <cstdio>
#include <type_traits>

#include "common.cuh"
#include "gist_internal.h"

namespace gist {

namespace {

template <int VEC>
struct VecT;
template <>
struct VecT<1> { using T = float; };
template <>
struct VecT<2> { using T = float2; };
template <>
struct VecT<4> { using T = float4; };

template <int VEC>
__device__ __forceinline__ void load_vec(const float* p, float (&x)[VEC]) {
  using T = typename VecT<VEC>::T;
  T v = *reinterpret_cast<const T*>(p);
  if constexpr (VEC == 1) {
    x[0] = v;
  } else if constexpr (VEC == 2) {
    x[0] = v.x; x[1] = v.y;
  } else {
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
  }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&x)[VEC]) {
  using T = typename VecT<VEC>::T;
  T v;
  if constexpr (VEC == 1) {
    v = x[0];
  } else if constexpr (VEC == 2) {
    v.x = x[0]; v.y = x[1];
  } else {
    v.x = x[0]; v.y = x[1]; v.z = x[2]; v.w = x[3];
  }
  *reinterpret_cast<T*>(p) = v;
}

// Rows with more entries than this are split: a wave's gathers of one row are
// a serial chain of latencies (eight at a time, about 0.7 us), so a hub row
// of 1,234 entries alone kept one wave for 109 us on a 20,000-node power-law
// graph whose other rows took a few (512 columns; now 42 us for the call).
constexpr int kLongRow = 128;
constexpr int kSegs = 16;   // one for each lane group of a wave of the narrowest rows

// Part q of a long row's entries r0 .. r1: whole batches of eight.
__device__ __forceinline__ void segment(int r0, int r1, int q, int& b, int& e) {
  const unsigned len = static_cast<unsigned>(r1 - r0);
  const unsigned seg = (len + 8 * kSegs - 1) / (8 * kSegs) * 8;
  b = r0 + static_cast<int>(min(q * seg, len));
  e = r0 + static_cast<int>(min((q + 1) * seg, len));
}

// Row of slot s (of `slots` in a block): consecutive rows share a block, so
// that their common neighbours' rows meet in one CU's L1; with `apart` the rows
// of a block lie rblocks apart, so that the hubs of a degree-ordered graph
// fall into different blocks.
__device__ __forceinline__ int64_t row_of(int64_t rblock, int64_t rblocks, int s, int slots, bool apart) {
  return apart ? s * rblocks + rblock : rblock * slots + s;
}

// Whether the first or the last 64th of the rows holds more than four times
// its share of the entries: a graph ordered by degree (scalar loads of the
// same three words in every block).  On a 20,000-node power-law graph ordered
// by degree, rows apart take 17 us at 16 columns and 39 at 512, consecutive
// ones 61 and 88; on 1M nodes in clusters of 150 (10 entries per row) rows
// apart take 82 us at 8 columns and 1,800 at 512, consecutive ones 43 and 1,640.
__device__ __forceinline__ bool skewed(const int* __restrict__ rowptr, int n) {
  const int64_t total = rowptr[n], slice = n / 64;
  return 16 * static_cast<int64_t>(rowptr[slice]) > total ||
         16 * (total - rowptr[n - slice]) > total;
}

template <int VEC, int LPR>
__global__ __launch_bounds__(256) void spmm_kernel(
    int n, const int* __restrict__ rowptr, const int* __restrict__ col,
    const float* __restrict__ val, const float* __restrict__ X, int64_t ldx, int width,
    float* Y, int64_t ldy, const float* add, int64_t ld_add, int relu, int col_tiles,
    int64_t nblocks, const float* mask, int64_t ldm, int spread) {
  constexpr int kWaves = 4;
  constexpr int RPW = 64 / LPR;  // rows per wave
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int grp = lane / LPR;       // row slot inside the wave
  const int gl = lane % LPR;        // lane inside the row group
  const int64_t logical = xcd_remap(blockIdx.x, nblocks);
  // column tile major: an XCD's contiguous range of blocks covers all rows
  // of one or a few column slabs, whose gathered rows then fit its L2
  const int64_t rblocks = nblocks / col_tiles;
  const int ctile = static_cast<int>(logical / rblocks);
  const int64_t rblock = logical - static_cast<int64_t>(ctile) * rblocks;
  const int64_t row = row_of(rblock, rblocks, wave * RPW + grp, kWaves * RPW, spread && skewed(rowptr, n));
  const int c0 = ctile * (LPR * VEC) + gl * VEC;
  const bool incol = c0 < width;
  const bool active = row < n && incol;

  int e0 = 0, e1 = 0;
  if (row < n) {
    e0 = rowptr[row];
    e1 = rowptr[row + 1];
  }
  // The epilogue's Add and mask values load before the row's gathers, so
  // their latency overlaps them (row and column clamped into the matrix:
  // every load is in bounds; an inactive lane's values are never stored).
  float a[VEC], mv[VEC];
  {
    const int64_t rr = min(row, static_cast<int64_t>(n) - 1);
    const int cc = min(c0, width - VEC);
    if (add) load_vec<VEC>(add + rr * ld_add + cc, a);
    if (mask) load_vec<VEC>(mask + rr * ldm + cc, mv);
  }
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;

  // Adds the entries base .. base + cnt (1 <= cnt <= LPR, the same for the whole
  // group) to acc: lane gl of the group loads one, then the group reads them
  // back by shuffle, four gathers in flight.
  auto window = [&](float (&acc)[VEC], int base, int cnt) {
    int my_c = 0;
    float my_v = 0.f;
    if (gl < cnt) {
      my_c = col[base + gl];
      my_v = val[base + gl];
    }
    int j = 0;
    for (; j + 4 <= cnt; j += 4) {
      int cj[4];
      float vj[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cj[u] = __shfl(my_c, grp * LPR + j + u, 64);
        vj[u] = __shfl(my_v, grp * LPR + j + u, 64);
      }
      if (incol) {
        float x[4][VEC];
#pragma unroll
        for (int u = 0; u < 4; ++u) load_vec<VEC>(X + static_cast<int64_t>(cj[u]) * ldx + c0, x[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] = fmaf(vj[u], x[u][v], acc[v]);
      }
    }
    if (j < cnt) {   // the rest together: loads past cnt repeat the last entry, not added
      int cj[3];
      float vj[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int k = grp * LPR + min(j + u, cnt - 1);
        cj[u] = __shfl(my_c, k, 64);
        vj[u] = __shfl(my_v, k, 64);
      }
      if (incol) {
        float x[3][VEC];
#pragma unroll
        for (int u = 0; u < 3; ++u) load_vec<VEC>(X + static_cast<int64_t>(cj[u]) * ldx + c0, x[u]);
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] = j + u < cnt ? fmaf(vj[u], x[u][v], acc[v]) : acc[v];
      }
    }
  };
  const bool is_long = RPW > 1 && e1 - e0 > kLongRow;
  {
    const int end = is_long ? e0 : e1;
    for (int base = e0; base < end; base += LPR) window(acc, base, min(LPR, end - base));
  }
  if constexpr (RPW > 1) {
    static_assert(kSegs % RPW == 0, "");
    // long rows: the wave's groups take the parts in turn
    unsigned long long todo = __ballot(is_long && gl == 0);
    while (todo) {
      const int owner = __ffsll(todo) - 1;
      todo &= todo - 1;
      const int l0 = __shfl(e0, owner, 64), l1 = __shfl(e1, owner, 64);
#pragma unroll 1
      for (int p = 0; p < kSegs; p += RPW) {
        float part[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) part[v] = 0.f;
        int b, e;
        segment(l0, l1, p + grp, b, e);
        for (int base = b; base < e; base += LPR) window(part, base, min(LPR, e - base));
#pragma unroll 2
        for (int q = 0; q < RPW; ++q)
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            const float x = __shfl(part[v], q * LPR + gl, 64);
            acc[v] = owner / LPR == grp ? acc[v] + x : acc[v];
          }
      }
    }
  }
  if (!active) return;
  if (add) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += a[v];
  }
  if (relu) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = fmaxf(acc[v], 0.f);
  }
  if (mask) {   // the ReLU derivative of the layer whose output is `mask`
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = mv[v] > 0.f ? acc[v] : 0.f;
  }
  store_vec<VEC>(Y + row * ldy + c0, acc);
}

// Wide rows (64 lanes per row): the row index is wave-uniform, so each
// nonzero's (col, val) is broadcast with readlane into scalar registers and
// the gather address is a scalar base plus the lane's column offset; eight
// gathers are kept in flight per wave.  A long row's parts are shared by the
// block's W waves.
template <int VEC, int W, bool SPREAD>
__global__ __launch_bounds__(64 * W) void spmm_wide_kernel(
    int n, const int* __restrict__ rowptr, const int* __restrict__ col,
    const float* __restrict__ val, const float* __restrict__ X, int64_t ldx, int width,
    float* Y, int64_t ldy, const float* add, int64_t ld_add, int relu, int col_tiles,
    int64_t nblocks, const float* mask, int64_t ldm) {
  __shared__ float part[kSegs][64 * VEC];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t logical = xcd_remap(blockIdx.x, nblocks);
  // column tile major: an XCD's contiguous range of blocks covers all rows
  // of one or a few column slabs, whose gathered rows then fit its L2
  const int64_t rblocks = nblocks / col_tiles;
  const int ctile = static_cast<int>(logical / rblocks);
  const int64_t rblock = logical - static_cast<int64_t>(ctile) * rblocks;
  const int c0 = ctile * (64 * VEC) + lane * VEC;
  const bool active = c0 < width;
  // lane w holds the extent of the block's row w, in every wave, so the whole
  // block knows the long ones without a barrier; with SPREAD lane W + w holds
  // that of its row in the other placement, so that neither load waits
  int s0 = 0, s1 = 0;
  {
    const int64_t r = row_of(rblock, rblocks, lane % W, W, SPREAD && (lane & W));
    if (r < n) {
      s0 = rowptr[r];
      s1 = rowptr[r + 1];
    }
  }
  const bool apart = SPREAD && skewed(rowptr, n);
  const int64_t row = row_of(rblock, rblocks, wave, W, apart);
  const bool inrow = row < n;
  if (SPREAD && apart) {
    s0 = __shfl(s0, lane | W, 64);
    s1 = __shfl(s1, lane | W, 64);
  }
  const unsigned longs = static_cast<unsigned>(__ballot(lane < W && s1 - s0 > kLongRow));
  int e0 = 0, e1 = 0;
  if (!(longs >> wave & 1)) {
    e0 = __builtin_amdgcn_readlane(s0, wave);
    e1 = __builtin_amdgcn_readlane(s1, wave);
  }
  // Add and mask values load before the gathers (row and column clamped into
  // the matrix: every load is in bounds; an inactive lane's values are never stored)
  float a[VEC], mv[VEC];
  {
    const int cc = min(c0, width - VEC);
    const int64_t rr = inrow ? row : n - 1;
    if (add) load_vec<VEC>(add + rr * ld_add + cc, a);
    if (mask) load_vec<VEC>(mask + rr * ldm + cc, mv);
  }
  const float* Xc = X + c0;
  float acc[VEC];
  // acc = the sum over entries e0 .. e1
  auto gather = [&](int e0, int e1) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    for (int base = e0; base < e1; base += 64) {
      const int cnt = min(64, e1 - base);
      int my_c = 0;
      float my_v = 0.f;
      if (lane < cnt) {
        my_c = col[base + lane];
        my_v = val[base + lane];
      }
      // U gathers in flight
      auto batch = [&](auto unroll, int j) {
        constexpr int U = decltype(unroll)::value;
        int cj[U];
        float vj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          cj[u] = __builtin_amdgcn_readlane(my_c, j + u);
          vj[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_v), j + u));
        }
        if (active) {
          float x[U][VEC];
#pragma unroll
          for (int u = 0; u < U; ++u) load_vec<VEC>(Xc + static_cast<int64_t>(cj[u]) * ldx, x[u]);
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = fmaf(vj[u], x[u][v], acc[v]);
        }
      };
      int j = 0;
      for (; j + 8 <= cnt; j += 8) batch(std::integral_constant<int, 8>{}, j);
      if (j + 4 <= cnt) {
        batch(std::integral_constant<int, 4>{}, j);
        j += 4;
      }
      if (j + 3 == cnt) batch(std::integral_constant<int, 3>{}, j);
      else if (j + 2 == cnt) batch(std::integral_constant<int, 2>{}, j);
      else if (j + 1 == cnt) batch(std::integral_constant<int, 1>{}, j);
    }
  };
  gather(e0, e1);
  if (longs) {
    float keep[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) keep[v] = acc[v];
    for (int w = 0; w < W; ++w) {
      if (!(longs >> w & 1)) continue;
      const int r0 = __builtin_amdgcn_readlane(s0, w), r1 = __builtin_amdgcn_readlane(s1, w);
      for (int q = wave; q < kSegs; q += W) {
        int b, e;
        segment(r0, r1, q, b, e);
        gather(b, e);
#pragma unroll
        for (int v = 0; v < VEC; ++v) part[q][lane * VEC + v] = acc[v];
      }
      __syncthreads();
      if (wave == w) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          float sum = 0.f;
#pragma unroll
          for (int q = 0; q < kSegs; ++q) sum += part[q][lane * VEC + v];
          keep[v] = sum;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = keep[v];
  }
  if (!inrow) return;
  if (!active) return;
  if (add) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += a[v];
  }
  if (relu) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = fmaxf(acc[v], 0.f);
  }
  if (mask) {   // the ReLU derivative of the layer whose output is `mask`
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = mv[v] > 0.f ? acc[v] : 0.f;
  }
  store_vec<VEC>(Y + row * ldy + c0, acc);
}

template <int VEC, int LPR>
gist_status launch(hipStream_t st, int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* col,
                   const float* val, const float* X, int64_t ldx, int width, float* Y,
                   int64_t ldy, const float* add, int64_t ld_add, bool relu, const float* mask,
                   int64_t ldm) {
  // sparse matrices may have hubs: rows apart if they come first (see skewed), and
  // (wide rows) eight waves per block to share one: with four, 512 columns
  // of a 20,000-node power-law graph took 50 us instead of 40
  const int spread = nnz <= 16 * n ? 1 : 0;
  const int waves = LPR == 64 && spread ? 8 : 4;
  constexpr int RPW = 64 / LPR;
  const int col_tiles = (width + LPR * VEC - 1) / (LPR * VEC);
  const int64_t rblocks = (n + waves * RPW - 1) / (waves * RPW);
  const int64_t nblocks = rblocks * col_tiles;
  if (nblocks > INT32_MAX) return set_error(GIST_E_UNSUPPORTED, "spmm: grid too large");
  char name[32];
  snprintf(name, sizeof(name), "spmm_v%d_l%d", VEC, LPR);
  // algorithmic bytes: rowptr, (col, val) per nonzero, X read once, Y written
  // once (and Add read once)
  const double bytes = 4.0 * (n + 1) + 8.0 * static_cast<double>(nnz) +
                       4.0 * static_cast<double>(n) * width * (2.0 + (add ? 1.0 : 0.0) +
                                                                (mask ? 1.0 : 0.0));
  ProfScope ps(st, name, 2.0 * static_cast<double>(nnz) * width, bytes);
  if constexpr (LPR == 64) {
    if (spread)
      hipLaunchKernelGGL((spmm_wide_kernel<VEC, 8, true>), dim3(static_cast<unsigned>(nblocks)), dim3(512),
                         0, st, static_cast<int>(n), rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu ? 1 : 0, col_tiles, nblocks, mask, ldm);
    else
      hipLaunchKernelGGL((spmm_wide_kernel<VEC, 4, false>), dim3(static_cast<unsigned>(nblocks)), dim3(256),
                         0, st, static_cast<int>(n), rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu ? 1 : 0, col_tiles, nblocks, mask, ldm);
  } else {
    hipLaunchKernelGGL((spmm_kernel<VEC, LPR>), dim3(static_cast<unsigned>(nblocks)), dim3(256),
                       0, st, static_cast<int>(n), rowptr, col, val, X, ldx, width, Y, ldy, add,
                       ld_add, relu ? 1 : 0, col_tiles, nblocks, mask, ldm, spread);
  }
  return check_launch("spmm");
}

template <int VEC>
gist_status launch_vec(hipStream_t st, int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* col,
                       const float* val, const float* X, int64_t ldx, int width, float* Y,
                       int64_t ldy, const float* add, int64_t ld_add, bool relu,
                       const float* mask, int64_t ldm) {
  // lanes per row: the smallest power of two covering the row, at most 64
  const int chunks = (width + VEC - 1) / VEC;
  if (chunks > 32)
    return launch<VEC, 64>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add, ld_add,
                               relu, mask, ldm);
  if (chunks > 16)
    return launch<VEC, 32>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add, ld_add,
                               relu, mask, ldm);
  if (chunks > 8)
    return launch<VEC, 16>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add, ld_add,
                               relu, mask, ldm);
  if (chunks > 4)
    return launch<VEC, 8>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add, ld_add,
                               relu, mask, ldm);
  return launch<VEC, 4>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add, ld_add,
                             relu, mask, ldm);
}

}  // namespace

gist_status spmm(hipStream_t st, int64_t n, int64_t nnz, const int32_t* rowptr, const int32_t* col,
                 const float* val, const float* X, int64_t ldx, int width, float* Y,
                 int64_t ldy, const float* add, int64_t ld_add, bool relu, const float* mask,
                 int64_t ldm) {
  if (n <= 0 || width <= 0) return GIST_OK;
  const bool v4 = width % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && aligned16(X) &&
                  aligned16(Y) && (!add || (ld_add % 4 == 0 && aligned16(add))) &&
                  (!mask || (ldm % 4 == 0 && aligned16(mask)));
  const bool v2 = width % 2 == 0 && ldx % 2 == 0 && ldy % 2 == 0 && aligned8(X) &&
                  aligned8(Y) && (!add || (ld_add % 2 == 0 && aligned8(add))) &&
                  (!mask || (ldm % 2 == 0 && aligned8(mask)));
  // Prefer the widest vector that still fills a 64-lane row; a row that
  // would need fewer than 33 lanes at 16 bytes uses 8-byte vectors instead
  // when that gives a full-wave row (e.g. width 100: 50 lanes x 2 floats).
  if (v4 && (width > 128 || width <= 64))
    return launch_vec<4>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu, mask, ldm);
  if (v2) return launch_vec<2>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu, mask, ldm);
  if (v4) return launch_vec<4>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu, mask, ldm);
  return launch_vec<1>(st, n, nnz, rowptr, col, val, X, ldx, width, Y, ldy, add,
                         ld_add, relu, mask, ldm);
}

}  // namespace gist
