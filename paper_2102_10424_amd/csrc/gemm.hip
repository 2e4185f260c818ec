// Dense contractions of the sub-GCN layer on the bf16 matrix cores.
//
// C (M x N) = act(A (M x K) * B (K x N)) for the three products of eq. (2)
// and its backward pass: the forward transform (Abar H) W (for GraphSAGE
// [H | Abar H] [W_self; W_neigh]), the weight gradient (Abar H)^T dZ and the
// input gradient dZ W^T.  Operands are read straight from the row-major
// activations and weights in whichever orientation the product needs.
//
// fp32 products, exact to fp32 level: a float has 24 significant bits, so it
// is the exact sum of three bf16 numbers, hi = bf16(x), mid = bf16(x - hi),
// lo = bf16(x - hi - mid), each rounded to nearest (both differences are
// exact).  The last bit of a float can be 2^-149, so both operands are split
// times 2^24 and the sums divided by 2^48 (both exact): no part is then a
// subnormal bf16 number.  (Unscaled, values below 2^-109 lost bits, and all of
// them below 2^-134.  2^16 would keep every bit, but the unit aligns a
// subnormal's products by its unnormalised exponent, which cost values below
// 2^-142 up to seven bits.)  A product is then
//   a b = hi hi' + hi mid' + mid hi' + hi lo' + mid mid' + lo hi' + (terms
//   below 2^-25 |a b| each),
// six bf16 products accumulated in fp32 by v_mfma_f32_32x32x16_bf16.  The
// bf16 unit multiplies 16 times as fast as the fp32 one, so six products
// still have 2.7 times its rate (419 against 157 TFLOP/s).  The split is made
// in registers on the way to LDS, so every value is split once per tile that
// uses it and memory sees the fp32 operands only.
//
// What bounds it: power, and beside it the vector unit (splitting, and the
// additions of gemm_split_kernel).  A loop of nothing but these MFMAs on random
// data holds 1,720 TFLOP/s (287 of fp32 products) at 1.8 GHz, on zeros 2,440; the
// 256 x 256 tiles keep the matrix cores busy 55-58% of the cycles, the
// 128 x 128 ones 63%.  On the products of a 4,096-wide GraphSAGE layer with 1,630
// nodes (109 GFLOP each), the fp32 matrix instruction took 985 / 985 / 950 us
// (forward, dH, dW; back to back, hot: between other kernels all of these are
// 5-10% less) and this 605 / 590 / 555; for 512 x 512 weights and 20,000 nodes
// 134 -> 85; a 1,536 x 64 product over K = 602 27 -> 11.
//
// Non-finite and huge values: the split of an Inf or NaN, or of a value that is
// Inf in bf16 when scaled (from 2^104 on), leaves NaN in the tile, and sums
// from 2^80 on overflow; so a wave whose accumulators hold anything non-finite
// recomputes its block with the fp32 matrix instruction straight from memory.
// No other input takes that path.  It is slow: of the products of a 4,096-wide GCN
// layer with 1,630 nodes, one NaN in H takes the forward from 350 to 1,200 us and
// dW from 300 to 700 (one such column or row is in every tile row or column),
// W all NaN dH from 330 to 1,700 (fp32 instruction throughout: 515, 510 and 515).
//
// bf16-input products round the operands (nearest even) on the same way to LDS
// and take one product: gemm_bf16_kernel (256 x 256 tiles) and
// gemm_small_kernel<1, ...>.

// Work distribution: tiles are whole where there are enough of them.  The
// tiles of the last, partly filled round (or all, where K is beyond 4,096 and
// the parts fit kMaxPartBytes) are cut in K, all at the same steps, slice-major, so that the workgroups an
// XCD runs together share each K range's operand rows in L2; what is left of
// each tile is dealt out in runs of the same length.  Partial tiles go to
// the workspace and a second kernel sums them in K order: deterministic, and
// no workgroup ever waits on another.

#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "common.cuh"
#include "gist_internal.h"

namespace gist {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

// Tile id -> (tile_m, tile_n): column-major in bands of 8 tile rows, so the
// tiles an XCD runs together share B columns and a narrow band of A rows.
__device__ __forceinline__ void tile_coords_banded(int64_t t, int tiles_m, int tiles_n, int& tm,
                                                   int& tn) {
  constexpr int kBand = 8;
  const int band = static_cast<int>(t / (static_cast<int64_t>(kBand) * tiles_n));
  const int rows_in_band = min(kBand, tiles_m - band * kBand);
  const int64_t in_band = t - static_cast<int64_t>(band) * kBand * tiles_n;
  tm = band * kBand + static_cast<int>(in_band % rows_in_band);
  tn = static_cast<int>(in_band / rows_in_band);
}

// Workgroup barrier that orders LDS only: waits for this wave's LDS
// accesses, not its global loads, so prefetches stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int KS = 16;         // K per step: one bf16 MFMA
constexpr int kRunK = 4096;    // values of K accumulated before the sign turns (gemm_split_kernel)

// Scale of both operands of an fp32 product, and what takes it out of the sums.
constexpr float kScale = 16777216.f, kUnscale = 1.f / (kScale * kScale);

// Operand view: element (r, k) at p[r * ld + k] (K contiguous) or
// p[k * ld + r]; p1 takes over at the segment boundary (along K or rows).
struct SOp {
  const float* p0;
  const float* p1;
  int64_t ld;
  int64_t gs0, gs1;
};

struct SOut {
  float* c0;
  float* c1;
  int64_t ldc0, ldc1, c_split;
  int64_t gs0, gs1;
  const float* mask;
  int64_t ldm, gsm;
  float lr;
  int relu, sgd;
};

// Work of one product: tiles of all groups, the first `whole` of them one
// workgroup each; the others (`ragged` of them) cut at the same K steps:
// `full` slices of `ipw` steps, slice-major, and the `rem` steps left of
// every tile dealt out in runs of ipw.
struct SSched {
  int64_t tiles, whole, ragged;
  int64_t tpg;                 // tiles per group
  int tiles_m, tiles_n, tm0;   // tm0: tile rows of the first row segment
  int nk, nf0, nf;             // K steps in all; whole ones of the first K segment, of both
  int full, ipw, rem;
  int parts;                   // partial slots per ragged tile (0: nothing is split)
};

__device__ __forceinline__ unsigned pk_bf16(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2){a, b}, bf16x2));
}

// Four values into their NP bf16 planes.
template <int NP>
__device__ __forceinline__ void split4(const float (&x)[4], uintx2 (&pl)[NP]) {
  float r[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
  for (int p = 0; p < NP; ++p) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned u = pk_bf16(r[2 * h], r[2 * h + 1]);
      pl[p][h] = u;
      if (p + 1 < NP) {
        r[2 * h] -= __builtin_bit_cast(float, u << 16);
        r[2 * h + 1] -= __builtin_bit_cast(float, u & 0xffff0000u);
      }
    }
  }
}

// LDS tile of one operand: 16-K chunks, planes, then blocks of 32 rows:
// 16-byte pieces (8 K) q = 0, 1 of the 32 rows, 1 KB per block.  The order of
// the rows inside a block, which also depends on the chunk c, spreads the
// fragment reads (32 rows, one piece) and the 8-byte staging writes (lanes along
// K, or along the rows in steps of one, two or four) over the banks.
__device__ __forceinline__ int lds_slot(int r, int q) {
  return r ^ ((r >> 3) & 1) ^ (((r >> 4) & 1) << 1) ^ (q * 4);
}
__host__ __device__ constexpr int chunk_xor(int c) { return (((c & 1) << 1) | ((c >> 1) & 1)) * 16; }
template <int ROWS>
__device__ __forceinline__ int lds_off(int row, int q) {
  return (row >> 5) * 1024 + q * 512 + lds_slot(row & 31, q) * 16;
}
template <int ROWS>
constexpr int plane_bytes() { return ROWS * 32; }

// One operand's share of a K step, held in registers between its load and
// its split.  Groups of four consecutive K of one row, in load items:
//   K contiguous: one group, V = 4, 2 or 1 floats per load;
//   row contiguous: R rows by four K, one load of R floats per K, R = 4 or 2
//     where the alignment allows.
// The load path takes four lanes per clock whatever their width (a wave's
// 8-byte load took 19 clocks, its 16-byte load 20), so loads are as wide as
// they can be; steps of 16 K leave only eight floats per thread, hence R = 2.
template <int NP, bool KM, int V, int ROWS, int THR, int KW, typename OFF>
struct Stage {
  static constexpr int NG = ROWS * (KW / 4) / THR;     // groups per thread
  static constexpr int R = KM ? 1 : V >= 4 && KW >= 32 ? 4 : V >= 2 && NG >= 2 ? 2 : 1;
  static constexpr int GP = R;                         // groups per load item
  static constexpr int NI = NG / GP;
  float v[NG][4];
  OFF off[NI];

  __device__ __forceinline__ static void item(int t, int i, int& row, int& kk) {
    const int x = t + THR * i;
    constexpr int L = KW / 4;   // lanes per row
    if constexpr (KM) { row = t / L + (THR / L) * i; kk = 4 * (t % L); }
    else { row = R * (x % (ROWS / R)); kk = 4 * (x / (ROWS / R)); }
  }
  __device__ __forceinline__ void init(int64_t ld, int rows_left, int t) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int row, kk;
      item(t, i, row, kk);
      if constexpr (KM)
        off[i] = static_cast<OFF>(min(row, rows_left - 1)) * static_cast<OFF>(ld * 4) + 4 * kk;
      else
        off[i] = static_cast<OFF>(4 * min(row, rows_left - R)) +
                 static_cast<OFF>(kk) * static_cast<OFF>(ld * 4);
    }
  }
  // base: the step's first element of the tile's first row; klim >= 1 values
  // of K exist from there on.  A load past them (EDGE only) reads the last ones.
  template <bool EDGE>
  __device__ __forceinline__ void load(int i, const char* base, OFF ld4, int klim, int t) {
    {
      int row, kk;
      item(t, i, row, kk);
      if constexpr (KM) {
#pragma unroll
        for (int j = 0; j < 4; j += V) {
          const char* p = EDGE ? base + (off[i] + static_cast<OFF>(4 * (min(kk + j, klim - V) - kk)))
                               : base + off[i] + 4 * j;
          if constexpr (V == 4) {
            const floatx4 x = *reinterpret_cast<const floatx4*>(p);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[i][q] = x[q];
          } else if constexpr (V == 2) {
            const floatx2 x = *reinterpret_cast<const floatx2*>(p);
            v[i][j] = x[0];
            v[i][j + 1] = x[1];
          } else {
            v[i][j] = *reinterpret_cast<const float*>(p);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const char* p = EDGE ? base + (off[i] + static_cast<OFF>(min(kk + j, klim - 1) - kk) * ld4)
                               : base + j * static_cast<int64_t>(ld4) + off[i];
          if constexpr (R == 4) {
            const floatx4 x = *reinterpret_cast<const floatx4*>(p);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[4 * i + q][j] = x[q];
          } else if constexpr (R == 2) {
            const floatx2 x = *reinterpret_cast<const floatx2*>(p);
            v[2 * i][j] = x[0];
            v[2 * i + 1][j] = x[1];
          } else {
            v[i][j] = *reinterpret_cast<const float*>(p);
          }
        }
      }
    }
  }
  // split group g, times sg for fp32 products, into the planes of the LDS tile S
  // (EDGE: K values from klim on are zero)
  template <bool EDGE>
  __device__ __forceinline__ void store(char* S, int g, int klim, float sg, int t) const {
    int row, kk;
    item(t, g / GP, row, kk);
    if constexpr (R > 1) row += g % R;
    float x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = !EDGE || kk + j < klim ? v[g][j] : 0.f;
      if (NP > 1) x[j] *= sg;
    }
    uintx2 pl[NP];
    split4<NP>(x, pl);
    const int c = KW > 16 ? kk >> 4 : 0;
    char* d = S + c * (NP * plane_bytes<ROWS>()) + (lds_off<ROWS>(row, (kk >> 3) & 1) ^ chunk_xor(c)) +
              ((kk >> 2) & 1) * 8;
#pragma unroll
    for (int p = 0; p < NP; ++p) *reinterpret_cast<uintx2*>(d + p * plane_bytes<ROWS>()) = pl[p];
  }
};

__device__ __forceinline__ float* s_ptr(const SOut& C, int64_t row, int64_t col) {
  return col < C.c_split ? C.c0 + row * C.ldc0 + col : C.c1 + row * C.ldc1 + (col - C.c_split);
}
__device__ __forceinline__ void s_store(const SOut& C, int64_t row, int64_t col, float v) {
  if (C.relu) v = fmaxf(v, 0.f);
  if (C.mask && col < C.c_split && !(C.mask[row * C.ldm + col] > 0.f)) v = 0.f;
  float* p = s_ptr(C, row, col);
  if (C.sgd) v = fmaf(-C.lr, v, *p);
  *p = v;
}

// K step j: its first K, the K values it has and its segment.  The whole
// steps of both segments come first, then each segment's partial step.
template <int KW>
__device__ __forceinline__ void k_step(const SSched& S, int64_t K, int64_t ksplit, int j, int64_t& k0,
                                       int& klim, bool& second) {
  if (j < S.nf) {
    second = j >= S.nf0;
    k0 = second ? ksplit + static_cast<int64_t>(j - S.nf0) * KW : static_cast<int64_t>(j) * KW;
    klim = KW;
  } else {
    second = j > S.nf || ksplit % KW == 0;
    k0 = second ? K - (K - ksplit) % KW : ksplit - ksplit % KW;
    klim = static_cast<int>((second ? K : ksplit) - k0);
  }
}

// The (tile, K range) runs of one workgroup.
struct Units {
  int64_t tile = 0;
  int kb = 0, ke = 0, part = 0;
  int64_t it = 0, it_end = 0;      // remainder region: over (ragged tile, remaining step)
  bool one = false, remainder = false;

  __device__ __forceinline__ explicit Units(const SSched& S) {
    const int64_t w = blockIdx.x;
    if (w < S.whole) {
      tile = xcd_remap(w, S.whole);
      ke = S.nk;
      one = true;
      return;
    }
    const int64_t u = xcd_remap(w - S.whole, gridDim.x - S.whole);
    const int64_t sliced = S.ragged * S.full;
    if (u < sliced) {
      part = static_cast<int>(u / S.ragged);
      tile = S.whole + (u - part * S.ragged);
      kb = part * S.ipw;
      ke = kb + S.ipw;
      one = true;
    } else {
      remainder = true;
      it = (u - sliced) * S.ipw;
      it_end = min(S.ragged * S.rem, it + S.ipw);
    }
  }
  __device__ __forceinline__ bool next(const SSched& S) {
    if (!remainder) {
      const bool r = one;
      one = false;
      return r;
    }
    if (it >= it_end) return false;
    const int64_t rt = it / S.rem;
    const int r0 = static_cast<int>(it - rt * S.rem);
    const int r1 = static_cast<int>(min<int64_t>(S.rem, r0 + (it_end - it)));
    tile = S.whole + rt;
    kb = S.full * S.ipw + r0;
    ke = S.full * S.ipw + r1;
    part = S.full + static_cast<int>(it / S.ipw - (rt * S.rem) / S.ipw);
    it += r1 - r0;
    return true;
  }
};

struct TilePos {
  int64_t grp, m0, mlim, n0;
  bool second;   // in the second row segment of A
};
template <int BM, int BN>
__device__ __forceinline__ TilePos tile_pos(const SSched& S, int64_t M, int64_t msplit, int64_t tile) {
  TilePos p;
  p.grp = tile / S.tpg;
  int tm, tn;
  tile_coords_banded(tile - p.grp * S.tpg, S.tiles_m, S.tiles_n, tm, tn);
  p.second = tm >= S.tm0;
  p.m0 = p.second ? msplit + static_cast<int64_t>(tm - S.tm0) * BM : static_cast<int64_t>(tm) * BM;
  p.mlim = p.second ? M : msplit;
  p.n0 = static_cast<int64_t>(tn) * BN;
  return p;
}

template <int WM, int WN>
__device__ __forceinline__ bool any_nonfinite(const floatx16 (&acc)[WM][WN]) {
  float z = 0.f;
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) z = fmaf(acc[a][b][r], 0.f, z);
  return __any(!(z == 0.f));
}

// This wave's block (rows wr.., columns wc.. of the tile, rows_left and
// cols_left in the tile) over K steps [kb, ke) on the fp32 matrix
// instruction, from memory.
template <int WM, int WN, int KW, bool AK, bool BK>
__device__ __forceinline__ void recompute(floatx16 (&acc)[WM][WN], const SSched& S, int64_t K, int64_t ksplit,
                                          int kb, int ke, const float* a0, const float* a1, int64_t lda,
                                          const float* b0, int64_t ldb, int wr, int wc, int64_t rows_left,
                                          int64_t cols_left) {
  const int li = threadIdx.x & 31, lh = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
  for (int j = kb; j < ke; ++j) {
    int64_t k0;
    int klim;
    bool second;
    k_step<KW>(S, K, ksplit, j, k0, klim, second);
    const float* pa = AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * lda;
    const float* pb = BK ? b0 + k0 : b0 + k0 * ldb;
    // Eight values of K at a time, four for each half of the wave.  (No faster
    // than two at a time, but the compiler then spills 32 instead of 112 vector
    // registers around the main loop of the 256 x 256 K x row-contiguous form.)
    for (int kk = 0; kk < klim; kk += 8) {
      float x[WM][4], y[WN][4];
#pragma unroll
      for (int a = 0; a < WM; ++a) {
        const int64_t r = min<int64_t>(wr + a * 32 + li, rows_left - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = min(kk + 4 * lh + i, klim - 1);
          x[a][i] = AK ? pa[r * lda + k] : pa[k * lda + r];
        }
      }
#pragma unroll
      for (int b = 0; b < WN; ++b) {
        const int64_t r = min<int64_t>(wc + b * 32 + li, cols_left - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = min(kk + 4 * lh + i, klim - 1);
          y[b][i] = BK ? pb[r * ldb + k] : pb[k * ldb + r];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = kk + 4 * lh + i < klim;
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? x[a][i] : 0.f, in ? y[b][i] : 0.f, acc[a][b],
                                                             0, 0, 0);
      }
    }
  }
}

// One 32 x 32 block to C.  Accumulator register r of lane l: row
// 8 (r / 4) + 4 (l / 32) + (r mod 4), column l mod 32.  The mask and the
// weights of a fused SGD step are all read before anything is written.
// WHOLE: all 32 rows lie in the matrix.  f: factor of the accumulators.
template <bool WHOLE>
__device__ __forceinline__ void store_block(const floatx16& acc, float f, const SOut& C, int64_t row0, int64_t mlim,
                                            int64_t col, int64_t N) {
  if (col >= N) return;
  const bool lo = col < C.c_split;
  const int64_t ld = lo ? C.ldc0 : C.ldc1;
  float* p = lo ? C.c0 + row0 * C.ldc0 + col : C.c1 + row0 * C.ldc1 + (col - C.c_split);
  const int left = static_cast<int>(min<int64_t>(mlim - row0, 32));
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = C.relu ? fmaxf(f * acc[r], 0.f) : f * acc[r];
  if (C.mask && lo) {
    const float* m = C.mask + row0 * C.ldm + col;
    float k[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = 8 * (r >> 2) + (r & 3);
      k[r] = WHOLE || rr < left ? m[rr * C.ldm] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = k[r] > 0.f ? v[r] : 0.f;
  }
  if (C.sgd) {
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = 8 * (r >> 2) + (r & 3);
      w[r] = WHOLE || rr < left ? p[rr * ld] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = fmaf(-C.lr, v[r], w[r]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rr = 8 * (r >> 2) + (r & 3);
    if (WHOLE || rr < left) p[rr * ld] = v[r];
  }
}

// This wave's block of a tile whose whole K it holds.
template <int WM, int WN>
__device__ __forceinline__ void store_tile(const floatx16 (&acc)[WM][WN], float f, const SOut& C, int64_t grp,
                                           int64_t row, int64_t mlim, int64_t col, int64_t N) {
  const int li = threadIdx.x & 31, lh = (threadIdx.x >> 5) & 1;
  SOut Cg = C;
  Cg.c0 += grp * C.gs0;
  Cg.c1 += grp * C.gs1;
  if (C.mask) Cg.mask += grp * C.gsm;
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b) {
      const int64_t r0 = row + a * 32 + 4 * lh, c = col + b * 32 + li;
      if (row + a * 32 + 32 <= mlim) store_block<true>(acc[a][b], f, Cg, r0, mlim, c, N);
      else store_block<false>(acc[a][b], f, Cg, r0, mlim, c, N);
    }
}

// A partial tile in accumulator order (block, r / 4, lane, r mod 4): 16-byte
// stores of whole lines.
template <int WM, int WN>
__device__ __forceinline__ void store_part(const floatx16 (&acc)[WM][WN], float f, float* part, int wave) {
  floatx4* dst = reinterpret_cast<floatx4*>(part) + wave * (WM * WN * 256) + (threadIdx.x & 63);
#pragma unroll
  for (int a = 0; a < WM; ++a)
#pragma unroll
    for (int b = 0; b < WN; ++b)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        floatx4 x;
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = f * acc[a][b][4 * r4 + q];
        dst[((a * WN + b) * 4 + r4) * 64] = x;
      }
}

// The fp32 product.  NWM x NWN waves of 32 WM x 32 WN blocks; 256 x 256 tiles
// by eight waves (one workgroup per CU) or 128 x 128 by four (two).  Every
// K step of 16 is 6 WM WN MFMAs per wave between two barriers; three LDS
// buffers of 6 bytes per value (144 KB at 256 x 256).  Larger tiles halve the
// splitting work and LDS traffic per MFMA (105 VALU for it to 48 MFMAs per wave
// and step at 256 x 256, twice that at 128 x 128), which is what is left of
// the power for the matrix cores.  Both use all 256 registers of two waves per
// SIMD: the compiler spills 20 to 40 vector registers around the main loop
// (the prologue and the epilogue), up to three accesses in it, and some 150
// scalar ones (the arguments) to vector lanes.
template <int WM, int WN, int NWM, int NWN, bool AK, bool BK, int V>
__global__ __launch_bounds__(64 * NWM * NWN, 2) void gemm_split_kernel(
    int64_t M, int64_t N, int64_t K, int64_t msplit, int64_t ksplit, SOp A, SOp B, SOut C, SSched S,
    float* __restrict__ partials) {
  constexpr int THR = 64 * NWM * NWN;
  constexpr int BM = 32 * WM * NWM, BN = 32 * WN * NWN;
  constexpr int ABYTES = 3 * plane_bytes<BM>(), BBYTES = 3 * plane_bytes<BN>();
  __shared__ __attribute__((aligned(16))) char lds[3][ABYTES + BBYTES];
  using SA = Stage<3, AK, V, BM, THR, KS, unsigned>;
  using SB = Stage<3, BK, V, BN, THR, KS, unsigned>;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int wm = wave / NWN, wn = wave % NWN;
  const int frag = lh * 512 + lds_slot(li, lh) * 16;   // this lane's chunk in a 32-row block

  Units units(S);
  // The large sums round as seldom as the registers allow (an instruction adds
  // its two halves of K in turn, so six in one chain round twelve times a
  // step, which on half-zero activations was more than the fp32 instruction).
  // Where they allow it the five small products have accumulators of their
  // own, added at the end: two roundings per step.  Else a block's products
  // of one step are summed from zero and added as one: one rounding, for 128
  // additions per wave and step.  Error of 4,096 cubed on ReLU activations:
  // 9.4e-7 in one chain, 3.2e-7 so (8.1e-7 on the fp32 instruction), and 578 /
  // 585 / 571 -> 639 / 636 / 632 us (KK, KR, RR).
  constexpr bool DUAL = WM * WN <= 4;
  floatx16 acc[WM][WN], low[DUAL ? WM : 1][DUAL ? WN : 1];
  SA sa;
  SB sb;
  while (units.next(S)) {
    const int kb = units.kb, ke = units.ke;
    const TilePos tp = tile_pos<BM, BN>(S, M, msplit, units.tile);
    const int64_t m0 = tp.m0, mlim = tp.mlim, n0 = tp.n0, grp = tp.grp;
    // first element of the tile's first row / column, per K segment
    const float *a0, *a1;
    if constexpr (AK) {
      a0 = A.p0 + grp * A.gs0 + m0 * A.ld;
      a1 = A.p1 + grp * A.gs1 + m0 * A.ld;
    } else {
      a0 = a1 = tp.second ? A.p1 + grp * A.gs1 + (m0 - msplit) : A.p0 + grp * A.gs0 + m0;
    }
    const float* b0 = B.p0 + grp * B.gs0 + (BK ? n0 * B.ld : n0);
    const unsigned lda4 = static_cast<unsigned>(A.ld * 4), ldb4 = static_cast<unsigned>(B.ld * 4);
    sa.init(A.ld, static_cast<int>(min<int64_t>(BM, mlim - m0)), t);
    sb.init(B.ld, static_cast<int>(min<int64_t>(BN, N - n0)), t);
    constexpr int NIT = SA::NI + SB::NI;   // load items per thread, A's first
    // The bf16 unit's sums round a little toward minus infinity (0.003 of a
    // unit in the last place per instruction, on average), which would add up
    // over a long K: every 4,096 values of K, and from one part of a tile to
    // the next, a workgroup turns from accumulating the product to its negative
    // or back (A negated on its way to LDS), so that the bias cancels.
    float sg = units.part & 1 ? -kScale : kScale;
    float f = units.part & 1 ? -kUnscale : kUnscale;   // takes sign and scale out of the sums
    struct Src { const char *a, *b; int klim; };
    auto src_full = [&](int j) {           // where whole step j is
      const bool second = j >= S.nf0;
      const int64_t k0 = static_cast<int64_t>(second ? j - S.nf0 : j) * KS + (second ? ksplit : 0);
      return Src{reinterpret_cast<const char*>(AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * A.ld),
                 reinterpret_cast<const char*>(BK ? b0 + k0 : b0 + k0 * B.ld), KS};
    };
    auto src_any = [&](int j) {
      int64_t k0;
      int klim;
      bool second;
      k_step<KS>(S, K, ksplit, j, k0, klim, second);
      return Src{reinterpret_cast<const char*>(AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * A.ld),
                 reinterpret_cast<const char*>(BK ? b0 + k0 : b0 + k0 * B.ld), klim};
    };
    auto load = [&](auto edge, int i, const Src& q) {
      constexpr bool E = decltype(edge)::value;
      if (i < SA::NI) sa.template load<E>(i, q.a, lda4, q.klim, t);
      else sb.template load<E>(i - SA::NI, q.b, ldb4, q.klim, t);
    };
    // split item i (its groups) into LDS buffer buf
    auto stage = [&](auto edge, int buf, int i, int klim) {
      constexpr bool E = decltype(edge)::value;
      if (i < SA::NI) {
#pragma unroll
        for (int g = 0; g < SA::GP; ++g) sa.template store<E>(lds[buf], i * SA::GP + g, klim, sg, t);
      } else {
#pragma unroll
        for (int g = 0; g < SB::GP; ++g)
          sb.template store<E>(lds[buf] + ABYTES, (i - SA::NI) * SB::GP + g, klim, kScale, t);
      }
    };
    constexpr std::true_type kEdge{};
    constexpr std::false_type kFull{};
    bf16x8 av[WM][3], bv[2][3];
    auto read_a = [&](int buf, int a, int p) {
      av[a][p] = *reinterpret_cast<const bf16x8*>(lds[buf] + (wm * WM + a) * 1024 + frag +
                                                  p * plane_bytes<BM>());
    };
    auto read_b = [&](int buf, int b, int p) {
      bv[b & 1][p] = *reinterpret_cast<const bf16x8*>(lds[buf] + ABYTES + (wn * WN + (b % WN)) * 1024 +
                                                      frag + p * plane_bytes<BN>());
    };
    // The six products of block column b, smallest first.  A's plane 2 is last
    // used by the first, its plane 1 by the third: `after` may then read the
    // next step's into those registers.
    constexpr int TA[6] = {2, 1, 1, 0, 0, 0}, TB[6] = {0, 1, 0, 2, 1, 0};
    auto mfmas = [&](int b, auto after) {
      if constexpr (DUAL) {
#pragma unroll
        for (int q = 0; q < 6; ++q) {
#pragma unroll
          for (int a = 0; a < WM; ++a) {
            floatx16& c = q < 5 ? low[a][b] : acc[a][b];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][TA[q]], bv[b & 1][TB[q]], c, 0, 0, 0);
          }
#pragma unroll
          for (int a = 0; a < WM; ++a) after(a, q);
        }
      } else {
        floatx16 c[WM] = {};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
#pragma unroll
          for (int a = 0; a < WM; ++a)
            c[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][TA[q]], bv[b & 1][TB[q]], c[a], 0, 0, 0);
#pragma unroll
          for (int a = 0; a < WM; ++a) after(a, q);
        }
#pragma unroll
        for (int a = 0; a < WM; ++a) acc[a][b] += c[a];
      }
    };
    // One K step from LDS buffer cur.  Every block of MFMAs also splits some
    // of step j + 2's items (in registers) into buffer free and at once
    // reloads them with step j + 3, so that a load has a whole step to
    // arrive; the last block reads the fragments that step j + 1 (in buffer
    // next, complete since the last barrier) starts with, so that its MFMAs
    // follow the barrier at once.
    auto step = [&](int cur, int next, int free, int jload) {
      const Src src = src_full(jload);
#pragma unroll
      for (int a = 0; a < WM; ++a) read_a(cur, a, 0);
#pragma unroll
      for (int b = 0; b < WN; ++b) {
#pragma unroll
        for (int p = 0; p < 3; ++p) read_b(b + 1 < WN ? cur : next, b + 1, p);
#pragma unroll
        for (int i = b * NIT / WN; i < (b + 1) * NIT / WN; ++i) {
          stage(kFull, free, i, KS);
          load(kFull, i, src);
        }
        mfmas(b, [&](int a, int q) {
          if (b == WN - 1 && (q == 0 || q == 2)) read_a(next, a, q == 0 ? 2 : 1);
        });
#pragma unroll
        for (int q = 0; q < 6 * WM; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an MFMA
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // some VALU
          __builtin_amdgcn_sched_group_barrier(0x080, 1, 0);   // an LDS access
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[a][b][r] = 0.f;
          if (DUAL) low[DUAL ? a : 0][DUAL ? b : 0][r] = 0.f;
        }

    // a wave wholly past the matrix only stages
    const bool live = wm * WM * 32 < mlim - m0 && wn * WN * 32 < N - n0;
    lds_barrier();   // the previous tile's LDS is consumed
    const int whole_end = min(ke, S.nf);
    for (int rb = kb; rb < whole_end; rb += kRunK / KS) {
      const int fe = min(rb + kRunK / KS, whole_end);
      if (rb > kb) {
        sg = -sg;
        f = -f;
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b) {
            acc[a][b] = -acc[a][b];
            if constexpr (DUAL) low[a][b] = -low[a][b];
          }
      }
      {
        Src q = src_full(rb);
#pragma unroll
        for (int i = 0; i < NIT; ++i) load(kFull, i, q);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          q = src_full(min(rb + s + 1, fe - 1));
#pragma unroll
          for (int i = 0; i < NIT; ++i) {
            stage(kFull, s, i, KS);
            load(kFull, i, q);
          }
        }
      }
      lds_barrier();
      int cur = 0, next = 1, free = 2;
      if (live) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          read_b(0, 0, p);
#pragma unroll
          for (int a = 0; a < WM; ++a) read_a(0, a, p);
        }
        for (int j = rb; j < fe; ++j) {
          step(cur, next, free, min(j + 3, fe - 1));
          lds_barrier();
          const int c = cur;
          cur = next;
          next = free;
          free = c;
        }
      } else {
        for (int j = rb; j < fe; ++j) {
          const Src q = src_full(min(j + 3, fe - 1));
#pragma unroll
          for (int i = 0; i < NIT; ++i) {
            stage(kFull, free, i, KS);
            load(kFull, i, q);
          }
          lds_barrier();
          const int c = cur;
          cur = next;
          next = free;
          free = c;
        }
      }
    }
    for (int j = max(kb, S.nf); j < ke; ++j) {   // the segments' partial steps
      const Src q = src_any(j);
#pragma unroll
      for (int i = 0; i < NIT; ++i) load(kEdge, i, q);
#pragma unroll
      for (int i = 0; i < NIT; ++i) stage(kEdge, 0, i, q.klim);
      lds_barrier();
      if (live) {
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int p = 0; p < 3; ++p) read_a(0, a, p);
#pragma unroll
        for (int b = 0; b < WN; ++b) {
#pragma unroll
          for (int p = 0; p < 3; ++p) read_b(0, b, p);
          mfmas(b, [](int, int) {});
        }
      }
      lds_barrier();
    }

    if constexpr (DUAL) {
#pragma unroll
      for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] += low[a][b];
    }
    if (any_nonfinite<WM, WN>(acc)) {
      f = 1.f;
      recompute<WM, WN, KS, AK, BK>(acc, S, K, ksplit, kb, ke, a0, a1, A.ld, b0, B.ld, wm * WM * 32,
                                    wn * WN * 32, mlim - m0, N - n0);
    }
    if (kb == 0 && ke == S.nk)
      store_tile<WM, WN>(acc, f, C, grp, m0 + wm * WM * 32, mlim, n0 + wn * WN * 32, N);
    else
      store_part<WM, WN>(acc, f,
                         partials + ((units.tile - S.whole) * S.parts + units.part) * static_cast<int64_t>(BM * BN),
                         wave);
  }
}

// Small products, and products with bf16 inputs (NP = 1: operands rounded to
// bf16, one product): four waves of 32 WM x 32 WN blocks, K steps of 64 so
// that a workgroup meets the memory latency once per 64 values of K.  One LDS
// tile (three workgroups per CU), the next step's loads in flight while this
// one multiplies.
constexpr int KL = 64;
template <int NP, int WM, int WN, bool AK, bool BK, int VA, int VB>
__global__ __launch_bounds__(256, WM == 1 ? 3 : 2) void gemm_small_kernel(
    int64_t M, int64_t N, int64_t K, int64_t msplit, int64_t ksplit, SOp A, SOp B, SOut C, SSched S,
    float* __restrict__ partials) {
  constexpr int BM = 64 * WM, BN = 64 * WN;
  constexpr int CA = NP * plane_bytes<BM>(), CB = NP * plane_bytes<BN>();   // bytes of 16 K
  __shared__ __attribute__((aligned(16))) char lds[(KL / 16) * (CA + CB)];
  using SA = Stage<NP, AK, VA, BM, 256, KL, int64_t>;
  using SB = Stage<NP, BK, VB, BN, 256, KL, int64_t>;
  constexpr bool EXACT = NP == 3;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int frag = (lane >> 5) * 512 + lds_slot(lane & 31, lane >> 5) * 16;
  char* const ldsB = lds + (KL / 16) * CA;
  floatx16 acc[WM][WN], low[EXACT ? WM : 1][EXACT ? WN : 1];   // low: the five small products
  SA sa;
  SB sb;
  Units units(S);
  while (units.next(S)) {
    const int kb = units.kb, ke = units.ke;
    const TilePos tp = tile_pos<BM, BN>(S, M, msplit, units.tile);
    const int64_t m0 = tp.m0, n0 = tp.n0, grp = tp.grp;
    const float *a0, *a1;
    if constexpr (AK) {
      a0 = A.p0 + grp * A.gs0 + m0 * A.ld;
      a1 = A.p1 + grp * A.gs1 + m0 * A.ld;
    } else {
      a0 = a1 = tp.second ? A.p1 + grp * A.gs1 + (m0 - msplit) : A.p0 + grp * A.gs0 + m0;
    }
    const float* b0 = B.p0 + grp * B.gs0 + (BK ? n0 * B.ld : n0);
    sa.init(A.ld, static_cast<int>(min<int64_t>(BM, tp.mlim - m0)), t);
    sb.init(B.ld, static_cast<int>(min<int64_t>(BN, N - n0)), t);
    auto load = [&](int j) {
      int64_t k0;
      int klim;
      bool second;
      k_step<KL>(S, K, ksplit, j, k0, klim, second);
      const char* pa = reinterpret_cast<const char*>(
          AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * A.ld);
      const char* pb = reinterpret_cast<const char*>(BK ? b0 + k0 : b0 + k0 * B.ld);
#pragma unroll
      for (int i = 0; i < SA::NI; ++i) sa.template load<true>(i, pa, A.ld * 4, klim, t);
#pragma unroll
      for (int i = 0; i < SB::NI; ++i) sb.template load<true>(i, pb, B.ld * 4, klim, t);
      return klim;
    };
    float sg = units.part & 1 ? -kScale : kScale;   // sg, f: see gemm_split_kernel
    float f = !EXACT ? 1.f : units.part & 1 ? -kUnscale : kUnscale;
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[a][b][r] = 0.f;
          if (EXACT) low[EXACT ? a : 0][EXACT ? b : 0][r] = 0.f;
        }
    int klim = load(kb);
    for (int j = kb; j < ke; ++j) {
      if (EXACT && j > kb && (j - kb) % (kRunK / KL) == 0) {
        sg = -sg;
        f = -f;
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b) {
            acc[a][b] = -acc[a][b];
            if constexpr (EXACT) low[a][b] = -low[a][b];
          }
      }
      lds_barrier();   // the last step's fragments are read
#pragma unroll
      for (int g = 0; g < SA::NG; ++g) sa.template store<true>(lds, g, klim, sg, t);
#pragma unroll
      for (int g = 0; g < SB::NG; ++g) sb.template store<true>(ldsB, g, klim, kScale, t);
      if (j + 1 < ke) klim = load(j + 1);
      lds_barrier();
#pragma unroll
      for (int c = 0; c < KL / 16; ++c) {
        bf16x8 av[WM][NP], bv[WN][NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
          for (int a = 0; a < WM; ++a)
            av[a][p] = *reinterpret_cast<const bf16x8*>(lds + c * CA + p * plane_bytes<BM>() +
                                                        (wm * WM + a) * 1024 + (frag ^ chunk_xor(c)));
#pragma unroll
          for (int b = 0; b < WN; ++b)
            bv[b][p] = *reinterpret_cast<const bf16x8*>(ldsB + c * CB + p * plane_bytes<BN>() +
                                                        (wn * WN + b) * 1024 + (frag ^ chunk_xor(c)));
        }
#pragma unroll
        for (int a = 0; a < WM; ++a)
#pragma unroll
          for (int b = 0; b < WN; ++b) {
            if constexpr (EXACT) {
              constexpr int TA[5] = {2, 1, 0, 1, 0}, TB[5] = {0, 1, 2, 0, 1};
#pragma unroll
              for (int q = 0; q < 5; ++q)
                low[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][TA[q]], bv[b][TB[q]], low[a][b], 0, 0, 0);
            }
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[a][0], bv[b][0], acc[a][b], 0, 0, 0);
          }
      }
    }
    if constexpr (EXACT) {
#pragma unroll
      for (int a = 0; a < WM; ++a)
#pragma unroll
        for (int b = 0; b < WN; ++b) acc[a][b] += low[a][b];
      if (any_nonfinite<WM, WN>(acc)) {
        f = 1.f;
        recompute<WM, WN, KL, AK, BK>(acc, S, K, ksplit, kb, ke, a0, a1, A.ld, b0, B.ld, wm * WM * 32,
                                      wn * WN * 32, tp.mlim - m0, N - n0);
      }
    }
    if (kb == 0 && ke == S.nk)
      store_tile<WM, WN>(acc, f, C, grp, m0 + wm * WM * 32, tp.mlim, n0 + wn * WN * 32, N);
    else
      store_part<WM, WN>(acc, f,
                         partials + ((units.tile - S.whole) * S.parts + units.part) * static_cast<int64_t>(BM * BN),
                         wave);
  }
}

// Large products with bf16 inputs: 256 x 256 tiles by eight waves of 64 x 128,
// K steps of 32, operands rounded to bf16 on the way to three LDS buffers.
// What bounds it: the fp32 operands, 64 KB per step and CU through the load
// path for 1,024 clocks of MFMAs per SIMD; that path is busy 70-80% of the
// kernel.  A wave's load takes 16 to 20 clocks there whatever its width, so
// both orientations load 16 bytes per lane: with 8-byte loads of a
// row-contiguous operand dW took 190 us instead of 156, with the two 16-byte
// halves of a lane's 32 bytes in turn (half lines) dH 167 instead of 150.
// On a 4,096-wide GraphSAGE layer with 1,630 nodes (109 GFLOP each; forward,
// dH, dW; back to back, hot): 209 / 167 / 206 us -> 202 / 150 / 156 (in a training
// round 165 / 141 / 158); four sub-GCNs' 3,100 x 1,024
// products over K = 2,048 in one grid instead of four: 340 -> 85 us.
constexpr int KB = 32;
template <bool AK, bool BK, int V>
__global__ __launch_bounds__(512, 2) void gemm_bf16_kernel(int64_t M, int64_t N, int64_t K, int64_t msplit,
                                                           int64_t ksplit, SOp A, SOp B, SOut C, SSched S,
                                                           float* __restrict__ partials) {
  constexpr int WM = 2, WN = 4, NWN = 2, THR = 512, BM = 256, BN = 256;
  constexpr int CA = plane_bytes<BM>(), CB = plane_bytes<BN>();   // bytes of 16 K
  __shared__ __attribute__((aligned(16))) char lds[3][2 * (CA + CB)];
  using SA = Stage<1, AK, V, BM, THR, KB, unsigned>;
  using SB = Stage<1, BK, V, BN, THR, KB, unsigned>;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / NWN, wn = wave % NWN;
  const int frag = (lane >> 5) * 512 + lds_slot(lane & 31, lane >> 5) * 16;
  floatx16 acc[WM][WN];
  SA sa;
  SB sb;
  Units units(S);
  while (units.next(S)) {
    const int kb = units.kb, ke = units.ke;
    const TilePos tp = tile_pos<BM, BN>(S, M, msplit, units.tile);
    const int64_t m0 = tp.m0, mlim = tp.mlim, n0 = tp.n0, grp = tp.grp;
    const float *a0, *a1;
    if constexpr (AK) {
      a0 = A.p0 + grp * A.gs0 + m0 * A.ld;
      a1 = A.p1 + grp * A.gs1 + m0 * A.ld;
    } else {
      a0 = a1 = tp.second ? A.p1 + grp * A.gs1 + (m0 - msplit) : A.p0 + grp * A.gs0 + m0;
    }
    const float* b0 = B.p0 + grp * B.gs0 + (BK ? n0 * B.ld : n0);
    const unsigned lda4 = static_cast<unsigned>(A.ld * 4), ldb4 = static_cast<unsigned>(B.ld * 4);
    sa.init(A.ld, static_cast<int>(min<int64_t>(BM, mlim - m0)), t);
    sb.init(B.ld, static_cast<int>(min<int64_t>(BN, N - n0)), t);
    constexpr int NIT = SA::NI + SB::NI;
    struct Src { const char *a, *b; int klim; };
    auto src = [&](int j) {
      int64_t k0;
      int klim;
      bool second;
      k_step<KB>(S, K, ksplit, j, k0, klim, second);
      return Src{reinterpret_cast<const char*>(AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * A.ld),
                 reinterpret_cast<const char*>(BK ? b0 + k0 : b0 + k0 * B.ld), klim};
    };
    auto src_full = [&](int j) {
      const bool second = j >= S.nf0;
      const int64_t k0 = static_cast<int64_t>(second ? j - S.nf0 : j) * KB + (second ? ksplit : 0);
      return Src{reinterpret_cast<const char*>(AK ? (second ? a1 + (k0 - ksplit) : a0 + k0) : a0 + k0 * A.ld),
                 reinterpret_cast<const char*>(BK ? b0 + k0 : b0 + k0 * B.ld), KB};
    };
    auto load = [&](auto edge, int i, const Src& q) {
      constexpr bool E = decltype(edge)::value;
      if (i < SA::NI) sa.template load<E>(i, q.a, lda4, q.klim, t);
      else sb.template load<E>(i - SA::NI, q.b, ldb4, q.klim, t);
    };
    auto stage = [&](auto edge, int buf, int i, int klim) {
      constexpr bool E = decltype(edge)::value;
      if (i < SA::NI) {
#pragma unroll
        for (int g = 0; g < SA::GP; ++g) sa.template store<E>(lds[buf], i * SA::GP + g, klim, 1.f, t);
      } else {
#pragma unroll
        for (int g = 0; g < SB::GP; ++g)
          sb.template store<E>(lds[buf] + 2 * CA, (i - SA::NI) * SB::GP + g, klim, 1.f, t);
      }
    };
    constexpr std::true_type kEdge{};
    constexpr std::false_type kFull{};
    bf16x8 av[2][WM], bv[2];   // A's fragments of both halves of a step; B's of this block and the next
    auto read_a = [&](int buf, int c, int a) {
      av[c][a] = *reinterpret_cast<const bf16x8*>(lds[buf] + c * CA + (wm * WM + a) * 1024 + (frag ^ chunk_xor(c)));
    };
    auto read_b = [&](int buf, int c, int b) {
      bv[b & 1] = *reinterpret_cast<const bf16x8*>(lds[buf] + 2 * CA + c * CB + (wn * WN + b) * 1024 + (frag ^ chunk_xor(c)));
    };
    auto mfmas = [&](int c, int b) {
#pragma unroll
      for (int a = 0; a < WM; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[c][a], bv[b & 1], acc[a][b], 0, 0, 0);
    };
    // One step: eight blocks of MFMAs (two halves of K, four block columns).
    // As in gemm_split_kernel, the items of step j + 2 go to LDS between them
    // and are at once reloaded with step j + 3, and the last block reads
    // the next step's first fragments before the barrier.
    auto step = [&](int cur, int next, int free, int jload) {
      const Src q = src_full(jload);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < WN; ++b) {
          const int blk = c * WN + b;
          if (b + 1 < WN) read_b(cur, c, b + 1);
          else read_b(c == 0 ? cur : next, c ^ 1, 0);
          if (b == WN - 2) {
#pragma unroll
            for (int a = 0; a < WM; ++a) read_a(c == 0 ? cur : next, c ^ 1, a);
          }
#pragma unroll
          for (int i = blk * NIT / (2 * WN); i < (blk + 1) * NIT / (2 * WN); ++i) {
            stage(kFull, free, i, KB);
            load(kFull, i, q);
          }
          mfmas(c, b);
#pragma unroll
          for (int x = 0; x < WM; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an MFMA
            __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);   // some VALU
            __builtin_amdgcn_sched_group_barrier(0x080, 2, 0);   // LDS accesses
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int a = 0; a < WM; ++a)
#pragma unroll
      for (int b = 0; b < WN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    const bool live = wm * WM * 32 < mlim - m0 && wn * WN * 32 < N - n0;
    lds_barrier();   // the previous tile's LDS is consumed
    const int fe = min(ke, S.nf);
    if (kb < fe) {
      {
        Src q = src_full(kb);
#pragma unroll
        for (int i = 0; i < NIT; ++i) load(kFull, i, q);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          q = src_full(min(kb + s + 1, fe - 1));
#pragma unroll
          for (int i = 0; i < NIT; ++i) {
            stage(kFull, s, i, KB);
            load(kFull, i, q);
          }
        }
      }
      lds_barrier();
      int cur = 0, next = 1, free = 2;
      if (live) {
        read_b(0, 0, 0);
#pragma unroll
        for (int a = 0; a < WM; ++a) read_a(0, 0, a);
        for (int j = kb; j < fe; ++j) {
          step(cur, next, free, min(j + 3, fe - 1));
          lds_barrier();
          const int c = cur;
          cur = next;
          next = free;
          free = c;
        }
      } else {   // a wave wholly past the matrix only stages
        for (int j = kb; j < fe; ++j) {
          const Src q = src_full(min(j + 3, fe - 1));
#pragma unroll
          for (int i = 0; i < NIT; ++i) {
            stage(kFull, free, i, KB);
            load(kFull, i, q);
          }
          lds_barrier();
          const int c = cur;
          cur = next;
          next = free;
          free = c;
        }
      }
    }
    for (int j = max(kb, S.nf); j < ke; ++j) {   // the segments' partial steps
      const Src q = src(j);
#pragma unroll
      for (int i = 0; i < NIT; ++i) load(kEdge, i, q);
#pragma unroll
      for (int i = 0; i < NIT; ++i) stage(kEdge, 0, i, q.klim);
      lds_barrier();
      if (live) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
          for (int a = 0; a < WM; ++a) read_a(0, c, a);
#pragma unroll
          for (int b = 0; b < WN; ++b) {
            read_b(0, c, b);
            mfmas(c, b);
          }
        }
      }
      lds_barrier();
    }
    if (kb == 0 && ke == S.nk)
      store_tile<WM, WN>(acc, 1.f, C, grp, m0 + wm * WM * 32, mlim, n0 + wn * WN * 32, N);
    else
      store_part<WM, WN>(acc, 1.f,
                         partials + ((units.tile - S.whole) * S.parts + units.part) * static_cast<int64_t>(BM * BN),
                         wave);
  }
}

// Sum of every ragged tile's partial tiles, in K order, and the epilogue.
// One float4 of the partials (four rows of a column) per thread; a wave's
// stores cover 128-byte runs of two rows.
template <int WM, int WN, int NWM, int NWN>
__global__ __launch_bounds__(256) void gemm_fixup(int64_t M, int64_t N, int64_t msplit, SSched S,
                                                        const float* __restrict__ partials, SOut C) {
  constexpr int BM = 32 * WM * NWM, BN = 32 * WN * NWN;
  const int64_t rt = blockIdx.x;
  const TilePos tp = tile_pos<BM, BN>(S, M, msplit, S.whole + rt);
  const int64_t mlim = tp.mlim, grp = tp.grp;
  const int e = blockIdx.y * 256 + threadIdx.x;
  const int lane = e & 63, r4 = (e >> 6) & 3, blk = e >> 8;
  const int wave = blk / (WM * WN), ab = blk % (WM * WN);
  const int64_t row = tp.m0 + ((wave / NWN) * WM + ab / WN) * 32 + 8 * r4 + 4 * (lane >> 5);
  const int64_t col = tp.n0 + ((wave % NWN) * WN + ab % WN) * 32 + (lane & 31);
  if (row >= mlim || col >= N) return;
  int parts = S.full;
  if (S.rem > 0)
    parts += static_cast<int>(((rt + 1) * S.rem - 1) / S.ipw - (rt * S.rem) / S.ipw) + 1;
  const floatx4* p = reinterpret_cast<const floatx4*>(partials + rt * S.parts * static_cast<int64_t>(BM * BN)) + e;
  floatx4 s = *p;
#pragma unroll 4
  for (int q = 1; q < parts; ++q) s += p[q * (BM * BN / 4)];
  SOut Cg = C;
  Cg.c0 += grp * C.gs0;
  Cg.c1 += grp * C.gs1;
  if (C.mask) Cg.mask += grp * C.gsm;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (row + q < mlim) s_store(Cg, row + q, col, s[q]);
}

// ---- host side ---------------------------------------------------------------

struct Cfg {
  int bm, bn, kw;     // tile, K per step
  int per_cu;         // workgroups a CU holds at once
  int min_steps;      // fewest steps worth a workgroup of their own
  int max_run;        // steps a workgroup accumulates at most, if the parts fit kMaxPartBytes
  double step_us;     // one step of one workgroup with per_cu of them on every CU
  double alone_us;    // the least a step takes (memory latency)
  double fixed_us;    // a workgroup's first loads and its stores
};
// 0..2: fp32; 3..5: bf16 inputs.  The times were measured with the machine full
// (256 x 256: 102 steps over 512 tiles in 550 us; 128 x 128: 102 steps over
// 2,048 tiles in 640; 64 x 64: 8 steps over 2,504 tiles in 112) and nearly
// empty; choose_cfg takes the shape whose estimate is lowest.  Where two
// are close: 300,000 x 256 over K = 256 takes 292 / 284 us with the two large
// fp32 tiles, 2,048 x 2,048 over K = 8,192 352 / 394; 3,100 x 1,024 over K = 1,204
// 72 / 73 / 89 with all three, 1,630 x 8,192 over K = 47 24 / 30 / 42, 2,000 x 128
// over K = 1,433 32 / 21 / 23, 3,100 x 64 over K = 602 35 / 21 / 12.
constexpr Cfg kCfg[] = {{256, 256, KS, 1, 8, kRunK / KS, 2.8, 1.65, 14.0},
                        {128, 128, KS, 2, 8, kRunK / KS, 1.5, 0.8, 7.0},
                        {64, 64, KL, 3, 2, kRunK / KL, 3.5, 1.0, 4.0},
                        {128, 128, 64, 2, 2, 1 << 20, 2.0, 1.0, 7.0},
                        {64, 64, 64, 3, 2, 1 << 20, 1.8, 0.8, 4.0},
                        {256, 256, 32, 1, 8, 1 << 20, 1.1, 0.9, 14.0}};
constexpr int64_t kCUs = 256;
constexpr unsigned threads_of(const Cfg& c) { return c.bm == 256 ? 512 : 256; }
constexpr int64_t kMaxLd = int64_t(1) << 22;   // 255 rows of it in 32 bits of bytes
// Parts of at most 4,096 values of K round less than longer ones, but hold
// M N K / 4,096 sums, twice the output and more for a product that has tiles
// enough: 80 GB for 2.45M x 4,096 over K = 8,192.  Beyond this much workspace K is
// cut only as far as the machine has to be filled (at most three parts for
// each workgroup it holds).
constexpr int64_t kMaxPartBytes = int64_t(256) << 20;

// Time of `units` workgroups of `steps` steps: whole rounds of full CUs,
// then a round with fewer workgroups on each CU.
double run_us(const Cfg& c, int64_t units, int steps) {
  const int64_t slots = kCUs * c.per_cu, rounds = units / slots, rest = units % slots;
  double us = rounds * (steps * c.step_us + c.fixed_us);
  if (rest > 0) {
    const double share = static_cast<double>((rest + kCUs - 1) / kCUs) / c.per_cu;
    us += steps * std::max(c.alone_us, c.step_us * share) + c.fixed_us;
  }
  return us;
}

SSched make_ssched(int64_t M, int64_t N, int64_t K, int64_t groups, int64_t msplit, int64_t ksplit,
                   const Cfg& c, double* cost) {
  SSched s{};
  s.tm0 = static_cast<int>((msplit + c.bm - 1) / c.bm);
  s.tiles_m = s.tm0 + static_cast<int>((M - msplit + c.bm - 1) / c.bm);
  s.tiles_n = static_cast<int>((N + c.bn - 1) / c.bn);
  s.nf0 = static_cast<int>(ksplit / c.kw);
  s.nf = s.nf0 + static_cast<int>((K - ksplit) / c.kw);
  s.nk = s.nf + (ksplit % c.kw != 0) + ((K - ksplit) % c.kw != 0);
  s.tpg = static_cast<int64_t>(s.tiles_m) * s.tiles_n;
  s.tiles = s.tpg * groups;
  s.whole = s.tiles;
  s.full = 1;
  s.ipw = s.nk;
  // K cut into parts of `ipw` steps (`most`: and no longer ones)
  auto cut = [&](int64_t tiles, int ipw, int most) {
    int full = s.nk / ipw, rem = s.nk - full * ipw;
    if (rem > 0 && (rem < c.min_steps / 2 || ipw == most)) {   // no sliver per tile; equal parts of a long K
      const int q = rem < c.min_steps / 2 && (s.nk + full - 1) / full <= most ? full : full + 1;
      ipw = (s.nk + q - 1) / q;
      full = s.nk / ipw;
      rem = s.nk - full * ipw;
    }
    s.ragged = tiles;
    s.whole = s.tiles - tiles;
    s.full = full;
    s.ipw = ipw;
    s.rem = rem;
    s.parts = full + (rem > 0 ? 2 : 0);
  };
  // time of writing and summing the parts
  auto fix_us = [&]() {
    return s.ragged ? 5.0 + 2.0 * s.ragged * (s.full + (s.rem > 0 ? 1.3 : 0.0)) * c.bm * c.bn * 4.0 / 5.0e6
                    : 0.0;
  };
  const int64_t slots = kCUs * c.per_cu;
  const int64_t waves = s.tiles / slots, r = s.tiles - waves * slots;
  auto units = [&]() {
    return s.ragged * s.full + (s.rem > 0 ? (s.ragged * s.rem + s.ipw - 1) / s.ipw : 0);
  };
  const SSched uncut = s;
  double us = 0.0;
  bool done = false;
  if (s.nk > c.max_run) {
    const int even = static_cast<int>(std::max<int64_t>((s.tiles * s.nk + slots - 1) / slots, c.min_steps));
    cut(s.tiles, std::min(even, c.max_run), c.max_run);
    us = run_us(c, units(), s.ipw) + fix_us();
    done = s.ragged * s.parts <= kMaxPartBytes / (int64_t(4) * c.bm * c.bn);
    if (!done) s = uncut;
  }
  if (!done) {
    us = run_us(c, s.tiles, s.nk);
    const int ipw = static_cast<int>(std::max<int64_t>((r * s.nk + slots - 1) / slots, c.min_steps));
    if (r > 0 && ipw < s.nk) {   // the last, partly filled round cut in K, if that is quicker
      cut(r, ipw, INT32_MAX);
      const double t = run_us(c, waves * slots, s.nk) + run_us(c, units(), s.ipw) + fix_us();
      if (t < us && s.ipw < s.nk) us = t;
      else s = uncut;
    }
  }
  if (cost) *cost = us;
  return s;
}

int64_t sgrid(const SSched& s) {
  return s.whole + s.ragged * s.full + (s.rem > 0 ? (s.ragged * s.rem + s.ipw - 1) / s.ipw : 0);
}

// Leading dimensions whose offsets inside a tile need more than 32 bits: only the
// small kernel, which has 64-bit ones, takes them.
bool far_ld(int64_t lda, int64_t ldb) { return lda >= kMaxLd || ldb >= kMaxLd; }

int choose_cfg(int64_t M, int64_t N, int64_t K, int dtype, int64_t groups, int64_t msplit, int64_t ksplit,
               bool far) {
  if (far) return dtype == GIST_DTYPE_BF16_IN ? 4 : 2;
  const int lo = dtype == GIST_DTYPE_BF16_IN ? 3 : 0, hi = dtype == GIST_DTYPE_BF16_IN ? 6 : 3;
  int best = lo;
  double bc = 1e300;
  for (int i = lo; i < hi; ++i) {
    double c;
    const SSched s = make_ssched(M, N, K, groups, msplit, ksplit, kCfg[i], &c);
    if (sgrid(s) > UINT32_MAX / threads_of(kCfg[i])) c += 1e200;   // a grid holds fewer than 2^32 threads
    if (c < bc) { bc = c; best = i; }
  }
  return best;
}

// Floats per load along the operand's contiguous dimension (4, 2 or 1).
int vec_of(const Operand& o, int64_t R, int64_t K) {
  const int64_t ext = o.k_major ? K : R;
  const int64_t sp = o.p1 ? o.split : ext;
  for (int v = 4; v > 1; v >>= 1) {
    const uintptr_t m = 4 * v - 1;
    if (o.ld0 % v == 0 && ext % v == 0 && sp % v == 0 && o.gs0 % v == 0 &&
        !(reinterpret_cast<uintptr_t>(o.p0) & m) &&
        (!o.p1 || (!(reinterpret_cast<uintptr_t>(o.p1) & m) && o.gs1 % v == 0)))
      return v;
  }
  return 1;
}

}  // namespace

size_t gemm_workspace(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int dtype, int64_t groups,
                      int64_t msplit, int64_t ksplit) {
  if (M <= 0 || N <= 0 || K <= 0 || groups <= 0) return 0;
  if (msplit <= 0) msplit = M;
  if (ksplit <= 0) ksplit = K;
  const Cfg& c = kCfg[choose_cfg(M, N, K, dtype, groups, msplit, ksplit, far_ld(lda, ldb))];
  const SSched s = make_ssched(M, N, K, groups, msplit, ksplit, c, nullptr);
  return static_cast<size_t>(s.ragged) * s.parts * c.bm * c.bn * sizeof(float);
}

gist_status gemm(hipStream_t st, int64_t M, int64_t N, int64_t K, const Operand& A, const Operand& B,
                 const GemmOut& C, int dtype, void* ws, size_t ws_bytes, int64_t groups) {
  if (M <= 0 || N <= 0 || groups <= 0) return GIST_OK;
  if (K <= 0) return set_error(GIST_E_UNSUPPORTED, "gemm: K == 0");
  const bool bf = dtype == GIST_DTYPE_BF16_IN;
  if (K > static_cast<int64_t>(INT32_MAX - 2) * KS)
    return set_error(GIST_E_UNSUPPORTED, "gemm: K too large");
  if ((!A.k_major && B.k_major) || (A.p1 && A.ld1 != A.ld0) || B.p1)
    return set_error(GIST_E_UNSUPPORTED, "gemm: operand form");
  const int64_t msplit = !A.k_major && A.p1 ? std::min(A.split, M) : M;
  const int64_t ksplit = A.k_major && A.p1 ? std::min(A.split, K) : K;
  const int ci = choose_cfg(M, N, K, dtype, groups, msplit, ksplit, far_ld(A.ld0, B.ld0));
  const Cfg& c = kCfg[ci];
  const SSched s = make_ssched(M, N, K, groups, msplit, ksplit, c, nullptr);
  const size_t need = static_cast<size_t>(s.ragged) * s.parts * c.bm * c.bn * sizeof(float);
  if (need > 0 && (!ws || ws_bytes < need))
    return set_error(GIST_E_NOMEM, "gemm: workspace too small");
  const int64_t grid = sgrid(s);
  if (grid > INT32_MAX || s.tiles > INT32_MAX) return set_error(GIST_E_UNSUPPORTED, "gemm: grid too large");
  SOp a{A.p0, A.p1 ? A.p1 : A.p0, A.ld0, A.gs0, A.p1 ? A.gs1 : A.gs0};
  SOp b{B.p0, B.p0, B.ld0, B.gs0, B.gs0};
  SOut o{C.c0, C.c1, C.ldc0, C.ldc1, C.c_split, C.gs0, C.gs1, C.mask, C.ldm, C.gsm, C.lr,
         C.relu ? 1 : 0, C.sgd ? 1 : 0};
  // floats per load: one width for both operands, except that the small
  // kernels keep 16-byte loads of one beside an odd-strided other (an output
  // layer's weights beside its activations: 37 -> 32 us for 47 classes over K = 8,192)
  int va = vec_of(A, M, K), vb = vec_of(B, N, K);
  if (c.kw != KL || (va > 1 && vb > 1)) va = vb = std::min(va, vb);
  else if (va == 2) va = 1;
  else if (vb == 2) vb = 1;
  float* part = static_cast<float*>(ws);
  {
    // variant name: dtype, the K-contiguous (K) / row-contiguous (R)
    // orientation of A and B, the tile, and the floats per load of each
    char name[48];
    snprintf(name, sizeof(name), "gemm_%s_%c%c_%dx%d_v%d%d", bf ? "bf16" : "f32", A.k_major ? 'K' : 'R',
             B.k_major ? 'K' : 'R', c.bm, c.bn, va, vb);
    const double md = static_cast<double>(M), nd = static_cast<double>(N), kd = static_cast<double>(K),
                 gd = static_cast<double>(groups);
    ProfScope ps(st, name, 2.0 * md * nd * kd * gd, 4.0 * (md * kd + kd * nd + md * nd) * gd);
    const dim3 g(static_cast<unsigned>(grid));
#define GIST_ARGS g, dim3(thr), 0, st, M, N, K, msplit, ksplit, a, b, o, s, part
#define GIST_LARGE(AK_, BK_, V_)                                                                             \
  do {                                                                                                       \
    if (ci == 0) hipLaunchKernelGGL((gemm_split_kernel<2, 4, 4, 2, AK_, BK_, V_>), GIST_ARGS);               \
    else if (ci == 1) hipLaunchKernelGGL((gemm_split_kernel<2, 2, 2, 2, AK_, BK_, V_>), GIST_ARGS);          \
    else hipLaunchKernelGGL((gemm_bf16_kernel<AK_, BK_, V_>), GIST_ARGS);                                    \
  } while (0)
#define GIST_SMALL(AK_, BK_, VA_, VB_)                                                                       \
  do {                                                                                                       \
    if (ci == 2) hipLaunchKernelGGL((gemm_small_kernel<3, 1, 1, AK_, BK_, VA_, VB_>), GIST_ARGS);            \
    else if (ci == 3) hipLaunchKernelGGL((gemm_small_kernel<1, 2, 2, AK_, BK_, VA_, VB_>), GIST_ARGS);       \
    else hipLaunchKernelGGL((gemm_small_kernel<1, 1, 1, AK_, BK_, VA_, VB_>), GIST_ARGS);                    \
  } while (0)
#define GIST_SPLIT_V(AK_, BK_)                            \
  do {                                                    \
    if (c.kw == KL) {                                     \
      if (va == 4 && vb == 4) GIST_SMALL(AK_, BK_, 4, 4); \
      else if (va == 4) GIST_SMALL(AK_, BK_, 4, 1);       \
      else if (vb == 4) GIST_SMALL(AK_, BK_, 1, 4);       \
      else if (va == 2) GIST_SMALL(AK_, BK_, 2, 2);       \
      else GIST_SMALL(AK_, BK_, 1, 1);                    \
    } else if (va == 4) GIST_LARGE(AK_, BK_, 4);          \
    else if (va == 2) GIST_LARGE(AK_, BK_, 2);            \
    else GIST_LARGE(AK_, BK_, 1);                         \
  } while (0)
    const unsigned thr = threads_of(c);
    if (A.k_major && B.k_major) GIST_SPLIT_V(true, true);
    else if (A.k_major) GIST_SPLIT_V(true, false);
    else GIST_SPLIT_V(false, false);
#undef GIST_SPLIT_V
#undef GIST_SMALL
#undef GIST_LARGE
#undef GIST_ARGS
  }
  {
    const gist_status r = check_launch("gemm");
    if (r != GIST_OK) return r;
  }
  if (s.ragged > 0) {
    ProfScope ps(st, "gemm_fixup", 0.0,
                 4.0 * s.ragged * static_cast<double>(c.bm) * c.bn * (s.full + 1.3 * (s.rem > 0) + 1.0));
    const dim3 g(static_cast<unsigned>(s.ragged), static_cast<unsigned>(c.bm * c.bn / 1024));
    if (c.bm == 256)
      hipLaunchKernelGGL((gemm_fixup<2, 4, 4, 2>), g, dim3(256), 0, st, M, N, msplit, s, part, o);
    else if (c.bm == 128)
      hipLaunchKernelGGL((gemm_fixup<2, 2, 2, 2>), g, dim3(256), 0, st, M, N, msplit, s, part, o);
    else
      hipLaunchKernelGGL((gemm_fixup<1, 1, 2, 2>), g, dim3(256), 0, st, M, N, msplit, s, part, o);
    return check_launch("gemm fix-up");
  }
  return GIST_OK;
}

}  // namespace gist
