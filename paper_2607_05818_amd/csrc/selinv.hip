// Full maps R_i = (G^-1)_ii by sparse-direct selected inversion.
//
// Block PCG pays one block solve per 64 nodes; a full map of a large stack
// needs every diagonal entry of G^-1, which a sparse Cholesky factorisation
// and the Takahashi recurrence give at the cost of a few factorisations.
// The symbolic part (nested dissection of the stacked grid, fronts, maps)
// is host code (selinv_plan.cpp); everything numeric runs here, in float64,
// level by level of the dissection tree (all fronts of one depth together).
//
// Factorisation (deepest level first): each front is a dense F x F
// column-major block over [pivots, update set Q].  Its lower triangle is
// gathered from the update matrices of its children and receives the entries
// of G in its pivot columns; what is above the diagonal is written before it
// is read.  Its k pivot columns are then eliminated 64 at a time, right-looking, as a
// block LDL^T: with P the panel and R every front row after it,
//   D_P = A_PP^-1 (in place of A_PP),  Lhat = A_RP D_P (kept transposed in
//   the unused upper block P x R),     A_RR -= Lhat A_RP^T  (lower).
// (the update for two panels at a time, the second panel's columns between).
// After the last panel the trailing Q x Q block is the update matrix passed
// to the parent.  (D_P and Lhat are all that the inversion reads, so neither
// a triangular factor of the panel nor its inverse is ever formed.)
//
// Selected inversion (roots first; Z = G^-1): a front first gathers Z_QQ
// from its parent's finished block, then takes its panels last to first.
// For a panel P with the rows R after it (the later pivots of the front and
// Q, all of whose Z entries are known by then):
//   Z_RP = -Z_RR Lhat,   Z_PP = D_P - Lhat^T Z_RP,
// the block form of the Takahashi identities, written over Lhat / A_RP / D_P
// in place (Z_RP, its transpose Z_PR, Z_PP).  The dense front makes the
// structure of every column the whole of R, so the supernodal block form
// applies to any panel split.  diag(Z_PP) is R_i for the panel's nodes.
//
// The dense work is 64 x 64 output tiles on the float64 matrix cores
// (v_mfma_f64_16x16x4); tiles of all fronts of a level share one launch
// (grid.y walks the fronts).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include "reff_internal.h"
#include "selinv_plan.h"
#include "tile_inverse.h"

namespace reff {
namespace {

constexpr int PT = 64;  // panel width and output tile edge
constexpr int LEAF_AREA = 16;
constexpr unsigned MAX_GY = 65535;

typedef double d4v __attribute__((ext_vector_type(4)));

// Device copy of a front (see SnFront), plus its per-level scratch slots.
struct DFront {
  int64_t off;   // arena offset of the F x F block
  int64_t poff;  // parent's arena offset, -1 at a root
  int64_t rel;   // into rel[]: F - k parent positions of Q
  int64_t piv;   // into piv_node[]: k node ids
  int64_t ybuf;  // offset of its F x 64 block in a K part's Y buffer
  int64_t part;  // offset of its row tiles' 64 x 64 partial products
  int64_t inv;   // into inv[]: pF positions within Q of its parent's rows, -1
  int32_t F, k, pF;
  int32_t child[2];  // -1: none with an update matrix
};

constexpr int KS = 32;  // K slice staged through LDS

// C(i, j) = alpha sum_{kk in [kb, ke)} A(i, kk) B(kk, j) [+ C(i, j) with ADD] on
// the 64 x 64 tile at (i0, j0) of an M x N column-major C (ldc).
//   A(i, kk) = TA ? A[i lda + kk] : A[kk lda + i]
//   B(kk, j) = TB ? B[kk ldb + j] : B[j ldb + kk]
//   C(i, j)  at TC ? C[i ldc + j] : C[j ldc + i]
// With LOWER, entries above the diagonal are not written.  Four waves;
// wave w owns tile rows 16 w .. 16 w + 15 as four 16 x 16 accumulators, each
// held with the lanes along C's contiguous index (for !TC the product is
// formed transposed): a load or store of C then covers whole 128-byte lines,
// four columns at a time, instead of 32 bytes in each of sixteen columns.
// K goes through LDS 32 at a time, the next slice's loads in flight (in
// registers) while the matrix cores work on the current one; with ADD the
// tile of C is loaded before the products (a panel step has only two slices,
// and the tile's latency would follow them otherwise).
template <bool TA, bool TB, bool TC, bool LOWER, bool ADD>
__device__ __forceinline__ void gemm_tile(int i0, int j0, int M, int N, int kb, int ke,
                                          double alpha, const double* A, int64_t lda,
                                          const double* B, int64_t ldb, double* C, int64_t ldc,
                                          double (*sA)[KS + 1], double (*sB)[PT + 1]) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int cc = lane & 15, kr = lane >> 4;
  d4v acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = d4v{0.0, 0.0, 0.0, 0.0};
  // Loads go through the slice's scalar base and 32-bit byte offsets.  Rows,
  // columns and K indices past the edge repeat the last one: entries past
  // the edge of C are not written, and past the end of K A is zeroed.
  const uint32_t la = 8u * (uint32_t)lda, lb = 8u * (uint32_t)ldb, lc = 8u * (uint32_t)ldc;
  const int mr = M - 1 - i0, nr = N - 1 - j0;
  double ra[8], rb[8];
  auto load = [&](int k0) {
    const char* pa = (const char*)(TA ? A + (int64_t)i0 * lda + k0 : A + (int64_t)k0 * lda + i0);
    const char* pb = (const char*)(TB ? B + (int64_t)k0 * ldb + j0 : B + (int64_t)j0 * ldb + k0);
    const int last = ke - 1 - k0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int ai = min(TA ? (t >> 5) + 8 * e : t & 63, mr);
      const int bj = min(TB ? t & 63 : (t >> 5) + 8 * e, nr);
      const int ak = TA ? t & 31 : (t >> 6) + 4 * e, bk = TB ? (t >> 6) + 4 * e : t & 31;
      const uint32_t ca = min(ak, last), cb = min(bk, last);
      const double va =
          *(const double*)(pa + (TA ? __umul24(ai, la) + 8u * ca : __umul24(ca, la) + 8u * ai));
      rb[e] = *(const double*)(pb + (TB ? __umul24(cb, lb) + 8u * bj : __umul24(bj, lb) + 8u * cb));
      ra[e] = ak <= last ? va : 0.0;
    }
  };
  char* pc = (char*)(TC ? C + (int64_t)i0 * ldc + j0 : C + (int64_t)j0 * ldc + i0);
  auto at = [&](int i, int j) -> double* {
    return (double*)(pc + (TC ? __umul24(i, lc) + 8u * j : __umul24(j, lc) + 8u * i));
  };
  // entry r of accumulator q within the tile
  auto row = [&](int r) { return 16 * w + (TC ? kr + 4 * r : cc); };
  auto col = [&](int q, int r) { return 16 * q + (TC ? cc : kr + 4 * r); };
  if (kb < ke) load(kb);
  double cv[4][4];
  if (ADD) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        cv[q][r] = *at(min(row(r), mr), min(col(q, r), nr));
  }
  for (int k0 = kb; k0 < ke; k0 += KS) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int idx = t + 256 * e;
      sA[TA ? idx >> 5 : idx & 63][TA ? idx & 31 : idx >> 6] = ra[e];
      sB[TB ? idx >> 6 : idx & 31][TB ? idx & 63 : idx >> 5] = rb[e];
    }
    __syncthreads();
    if (k0 + KS < ke) load(k0 + KS);
#pragma unroll
    for (int ks = 0; ks < KS / 4; ++ks) {
      const double av = sA[16 * w + cc][4 * ks + kr];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double bv = sB[4 * ks + kr][16 * q + cc];
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(TC ? av : bv, TC ? bv : av, acc[q], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = row(r), j = col(q, r);
      if (i <= mr && j <= nr && !(LOWER && i0 + i < j0 + j))
        *at(i, j) = ADD ? cv[q][r] + alpha * acc[q][r] : alpha * acc[q][r];
    }
}

__global__ void k_zero(double* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// Entries of G into the assembled fronts (each position occurs once).
__global__ void k_scatter_add(const int64_t* __restrict__ idx, const double* __restrict__ val,
                              int64_t n, double* __restrict__ ar) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    ar[idx[e]] += val[e];
}

// inv[f.inv + r] = a where rel[f.rel + a] = r, -1 for the parent's other rows.
__global__ __launch_bounds__(256) void k_invert_rel(const DFront* __restrict__ fr, int nf,
                                                    const int32_t* __restrict__ rel,
                                                    int32_t* __restrict__ inv) {
  for (int fi = blockIdx.x; fi < nf; fi += gridDim.x) {
    const DFront f = fr[fi];
    if (f.poff < 0) continue;
    for (int r = threadIdx.x; r < f.pF; r += 256) inv[f.inv + r] = -1;
    __syncthreads();
    for (int a = threadIdx.x; a < f.F - f.k; a += 256) inv[f.inv + rel[f.rel + a]] = a;
  }
}

// Assembly: the lower triangle of each front as the sum of its children's
// update matrices (their trailing (F-k) x (F-k) blocks), child 0 before 1.
// One wave per AC columns, its lanes down the rows: inv is increasing where
// it is not -1, so the children's columns are read in order, and every entry
// of the front is written once.  Bound by those bytes: 4 x 512 x 512 takes
// 2.7 ms, where clearing the fronts and adding the children into them one
// after the other read and wrote each entry up to three times (4.4 ms).
constexpr int AC = 4;

__global__ __launch_bounds__(256) void k_assemble(const DFront* __restrict__ fr,
                                                  const int32_t* __restrict__ list, int nf,
                                                  const int32_t* __restrict__ inv, double* ar) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
    const DFront f = fr[list[fi]];
    const int32_t* im[2] = {inv, inv};
    const double* u[2] = {ar, ar};
    int64_t uF[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (f.child[c] >= 0) {
        const DFront g = fr[f.child[c]];
        im[c] = inv + g.inv;
        u[c] = ar + g.off + (int64_t)g.k * g.F + g.k;
        uF[c] = g.F;
      }
    const bool has[2] = {f.child[0] >= 0, f.child[1] >= 0};
    for (int c0 = (blockIdx.x * 4 + w) * AC; c0 < f.F; c0 += gridDim.x * 4 * AC) {
      const double* col[2][AC];
      bool on[2][AC];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < AC; ++j) {
          const int b = has[c] ? im[c][min(c0 + j, f.F - 1)] : -1;
          on[c][j] = b >= 0 && c0 + j < f.F;
          col[c][j] = on[c][j] ? u[c] + b * uF[c] : u[c];
        }
      double* dst = ar + f.off + (int64_t)c0 * f.F;
      for (int r = c0 + lane; r < f.F; r += 64) {
        double v[AC];
#pragma unroll
        for (int j = 0; j < AC; ++j) v[j] = 0.0;
        // Every load is made, from the child's first update row where there
        // is nothing to add (a listed child has one): eight in flight per lane
        // instead of a branch each.
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (has[c]) {
            const int a = im[c][r];
            double x[AC];
#pragma unroll
            for (int j = 0; j < AC; ++j) x[j] = col[c][j][max(a, 0)];
#pragma unroll
            for (int j = 0; j < AC; ++j) v[j] += a >= 0 && on[c][j] ? x[j] : 0.0;
          }
#pragma unroll
        for (int j = 0; j < AC; ++j)
          if (r >= c0 + j && c0 + j < f.F) dst[(int64_t)j * f.F + r] = v[j];
      }
    }
  }
}

// Z_QQ of each front (full square) from its parent's finished block; one
// wave per column (four per workgroup, blockIdx.x walks the columns).
__global__ __launch_bounds__(256) void k_gather(const DFront* __restrict__ fr,
                                                const int32_t* __restrict__ list, int nf,
                                                const int32_t* __restrict__ rel, double* ar) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
    const DFront f = fr[list[fi]];
    if (f.poff < 0) continue;
    const int q = f.F - f.k;
    const int32_t* rl = rel + f.rel;
    for (int b = blockIdx.x * 4 + w; b < q; b += gridDim.x * 4) {
      double* dst = ar + f.off + (int64_t)(f.k + b) * f.F + f.k;
      const double* src = ar + f.poff + (int64_t)rl[b] * f.pF;
      for (int a = lane; a < q; a += 64) dst[a] = src[rl[a]];
    }
  }
}

// D_P = A_PP^-1 of panel jp of every front, in place (full square).
__global__ __launch_bounds__(256) void k_tile(const DFront* __restrict__ fr,
                                              const int32_t* __restrict__ list, int nf, int jp,
                                              double* ar, int* bad) {
  __shared__ double T[PT][PT + 1];
  const int t = threadIdx.x;
  for (int fi = blockIdx.x; fi < nf; fi += gridDim.x) {
    const DFront f = fr[list[fi]];
    const int j0 = PT * jp;
    if (f.k <= j0) continue;
    const int w = min(PT, f.k - j0);
    double* a = ar + f.off + (int64_t)j0 * f.F + j0;
#pragma unroll
    for (int e = t; e < PT * PT; e += 256) {
      const int r = e & 63, c = e >> 6;
      if (r < c) continue;
      const double v = r < w ? a[(int64_t)c * f.F + r] : (r == c ? 1.0 : 0.0);
      T[r][c] = v;
      T[c][r] = v;
    }
    __syncthreads();
    invert_tile(T, w, bad);
    for (int e = t; e < PT * PT; e += 256) {
      const int r = e & 63, c = e >> 6;
      if (r < w && c < w) a[(int64_t)c * f.F + r] = T[r][c];
    }
    __syncthreads();  // before the next front's loads
  }
}

enum GemmOp { OP_LHAT = 0, OP_UPDATE = 1, OP_Y = 2 };

__device__ __forceinline__ void lower_tile(int t, int& ti, int& tj) {
  ti = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  while (ti * (ti + 1) / 2 > t) --ti;
  tj = t - ti * (ti + 1) / 2;
}

// Update tiles of a front after panel jp, m rows left: the lower triangle
// after an odd panel or the last one, with the products of the panel before
// it too; after the others only the next panel's columns.  An update reads
// and writes every entry of the triangle for 64 products each, which is
// bound by those bytes: with two panels per pass the updates of
// 4 x 512 x 512 take 5.9 ms instead of 6.8.
__host__ __device__ inline int update_tiles(int F, int k, int jp) {
  const int r0 = PT * (jp + 1) < k ? PT * (jp + 1) : k, ntile = (F - r0 + PT - 1) / PT;
  return (jp & 1) == 0 && k > r0 ? ntile : ntile * (ntile + 1) / 2;
}

// The panel products of step jp for every front of a level (see the file
// comment); blockIdx.x is the tile (for OP_Y, with its part of the K range).
template <int OP>
__global__ __launch_bounds__(256, OP == OP_UPDATE ? 3 : 4) void k_front_gemm(const DFront* __restrict__ fr,
                                                    const int32_t* __restrict__ list, int nf,
                                                    int jp, double* ar, int tiles, int ysplit,
                                                    double* __restrict__ Ysp, int64_t ylev) {
  __shared__ double sA[PT][KS + 1], sB[KS][PT + 1];
  for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
    const DFront f = fr[list[fi]];
    const int j0 = PT * jp;
    if (f.k <= j0) continue;
    const int w = min(PT, f.k - j0), r0 = j0 + w, m = f.F - r0;
    const int64_t F = f.F;
    double* base = ar + f.off;
    double* a_rp = base + (int64_t)j0 * F + r0;  // lower block, A[row][panel column]
    double* lhat = base + (int64_t)r0 * F + j0;  // upper block: Lhat(i, p) at [i F + p]
    const int ntile = (m + PT - 1) / PT;
    if (OP == OP_LHAT) {
      if ((int)blockIdx.x >= ntile) continue;
      gemm_tile<false, false, true, false, false>(blockIdx.x * PT, 0, m, w, 0, w, 1.0, a_rp, F,
                                                  base + (int64_t)j0 * F + j0, F, lhat, F, sA, sB);
    } else if (OP == OP_UPDATE) {
      if ((int)blockIdx.x >= update_tiles(f.F, f.k, jp)) continue;
      const bool pair = (jp & 1) == 0 && f.k > r0;  // the next panel brings the rest
      int ti = blockIdx.x, tj = 0;
      if (!pair) lower_tile(blockIdx.x, ti, tj);
      const int before = jp & 1 ? PT : 0;  // columns of the panel before
      const int n = pair ? min(PT, f.k - r0) : m;
      gemm_tile<true, true, false, true, true>(ti * PT, tj * PT, m, n, 0, before + w, -1.0,
                                               lhat - before, F, a_rp - before * F, F,
                                               base + (int64_t)r0 * F + r0, F, sA, sB);
    } else {
      // Y = -Z_RR Lhat over A_RP; with ysplit > 1, the K range in ysplit
      // parts, each into its own Y buffer (summed by k_finish)
      const int tile = (int)blockIdx.x % tiles, sp = (int)blockIdx.x / tiles;
      if (tile >= ntile) continue;
      int kb = 0, ke = m;
      double* y = a_rp;
      if (ysplit > 1) {
        const int ks = ((m + ysplit - 1) / ysplit + KS - 1) / KS * KS;
        kb = min(m, sp * ks);
        ke = min(m, kb + ks);
        y = Ysp + (size_t)sp * ylev + f.ybuf;
      }
      gemm_tile<false, true, false, false, false>(tile * PT, 0, m, w, kb, ke, -1.0,
                                                  base + (int64_t)r0 * F + r0, F, lhat, F, y, F, sA,
                                                  sB);
    }
    __syncthreads();
  }
}

// End of a selected-inversion panel step.  Per 64-row tile of R: sums the
// K parts of Y, writes Z_RP = Y and Z_PR = Y^T (over Lhat^T, which only this
// workgroup still reads) and forms -Lhat^T Y.  WHOLE: one workgroup takes all
// row tiles of a front and finishes Z_PP = D_P - Lhat^T Y with diag(Z_PP) into
// Rfull (levels with enough fronts to fill the chip); otherwise blockIdx.x
// is the row tile and its product goes to `part` for k_zpp.  Bound by the
// bytes of Y and Lhat; at the root panels of the 4 x 512 x 512 stack 22 us with
// k_zpp, where separate launches for the sum of the K parts, the product and
// the write-back took 107 us.
template <bool WHOLE>
__global__ __launch_bounds__(256, 2) void k_finish(const DFront* __restrict__ fr,
                                                const int32_t* __restrict__ list, int nf, int jp,
                                                double* ar, int ysplit,
                                                const double* __restrict__ Ysp, int64_t ylev,
                                                double* __restrict__ part,
                                                const int64_t* __restrict__ piv_node,
                                                double* __restrict__ Rfull) {
  __shared__ double sL[PT][PT + 1], sY[PT][PT + 1];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int cc = lane & 15, kr = lane >> 4;
  for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
    const DFront f = fr[list[fi]];
    const int j0 = PT * jp;
    if (f.k <= j0) continue;
    const int w = min(PT, f.k - j0), r0 = j0 + w, m = f.F - r0;
    const int64_t F = f.F;
    double* base = ar + f.off;
    const int ntile = (m + PT - 1) / PT;
    d4v acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = d4v{0.0, 0.0, 0.0, 0.0};
    const int rt0 = WHOLE ? 0 : (int)blockIdx.x, rt1 = WHOLE ? ntile : min(rt0 + 1, ntile);
    for (int rt = rt0; rt < rt1; ++rt) {
      const int i0 = rt * PT, rows = min(PT, m - i0);
      char* y_rp = (char*)(base + (int64_t)j0 * F + r0 + i0);  // (row, p) at [p F + row]
      char* z_pr = (char*)(base + (int64_t)(r0 + i0) * F + j0);  // (p, row) at [row F + p]
      // Y: lane = row, wv + 4 e = panel column; Lhat: the reverse.  Byte
      // offsets from the scalar bases, clamped to the tile's edge.
      const uint32_t f8 = 8u * (uint32_t)F;
      auto oy = [&](int e) { return __umul24(min(wv + 4 * e, w - 1), f8) + 8u * min(lane, rows - 1); };
      auto ol = [&](int e) { return __umul24(min(wv + 4 * e, rows - 1), f8) + 8u * min(lane, w - 1); };
      double v[16];
      if (ysplit > 1) {
        const char* src = (const char*)(Ysp + f.ybuf + i0);
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = 0.0;
        for (int s = 0; s < ysplit; ++s, src += 8 * ylev)
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] += *(const double*)(src + oy(e));
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = *(const double*)(y_rp + oy(e));
      }
      __syncthreads();  // the previous tile's LDS reads are done
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sY[lane][wv + 4 * e] = lane < rows ? v[e] : 0.0;
        if (ysplit > 1 && lane < rows && wv + 4 * e < w) *(double*)(y_rp + oy(e)) = v[e];
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = *(const double*)(z_pr + ol(e));
#pragma unroll
      for (int e = 0; e < 16; ++e) sL[wv + 4 * e][lane] = v[e];
      __syncthreads();
      // entries past w repeat the last column and are not written
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (wv + 4 * e < rows && lane < w) *(double*)(z_pr + ol(e)) = sY[wv + 4 * e][lane];
#pragma unroll 4
      for (int ks = 0; ks < PT / 4; ++ks) {
        const double av = sL[4 * ks + kr][16 * wv + cc];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, sY[4 * ks + kr][16 * q + cc], acc[q],
                                                        0, 0, 0);
      }
    }
    if (WHOLE) {
      double* z = base + (int64_t)j0 * F + j0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * wv + kr + 4 * r, j = 16 * q + cc;
          if (i >= w || j >= w) continue;
          const double v = z[(int64_t)j * F + i] - acc[q][r];
          z[(int64_t)j * F + i] = v;
          if (i == j) Rfull[piv_node[f.piv + j0 + i]] = v;
        }
    } else if (rt0 < ntile) {
      double* pp = part + f.part + (int64_t)rt0 * PT * PT;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) pp[(16 * q + cc) * PT + 16 * wv + kr + 4 * r] = acc[q][r];
    }
    __syncthreads();
  }
}

// Z_PP = D_P - the row tiles' products, in order (blockIdx.x: a 1024-entry
// quarter of the tile), diag(Z_PP) into Rfull.
__global__ __launch_bounds__(256) void k_zpp(const DFront* __restrict__ fr,
                                             const int32_t* __restrict__ list, int nf, int jp,
                                             double* ar, const double* __restrict__ part,
                                             const int64_t* __restrict__ piv_node,
                                             double* __restrict__ Rfull) {
  for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
    const DFront f = fr[list[fi]];
    const int j0 = PT * jp;
    if (f.k <= j0) continue;
    const int w = min(PT, f.k - j0), m = f.F - j0 - w, ntile = (m + PT - 1) / PT;
    double* z = ar + f.off + (int64_t)j0 * f.F + j0;
    const double* pp = part + f.part + blockIdx.x * 1024 + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int s = 0; s < ntile; ++s, pp += PT * PT)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += pp[256 * e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int idx = blockIdx.x * 1024 + threadIdx.x + 256 * e, j = idx >> 6, i = idx & 63;
      if (i >= w || j >= w) continue;
      const double x = z[(int64_t)j * f.F + i] - v[e];
      z[(int64_t)j * f.F + i] = x;
      if (i == j) Rfull[piv_node[f.piv + j0 + i]] = x;
    }
  }
}

__global__ void k_pick(const double* __restrict__ Rfull, const int64_t* __restrict__ nodes,
                       int64_t n, double* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = Rfull[nodes[i]];
}

dim3 flat(int64_t n) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192))); }

struct Bufs {
  std::vector<void*> ptrs;
  ~Bufs() {
    for (void* p : ptrs) (void)hipFree(p);
  }
  template <typename T>
  hipError_t get(T** out, size_t count) {
    void* p = nullptr;
    ptrs.reserve(ptrs.size() + 1);
    hipError_t e = hipMalloc(&p, std::max<size_t>(count, 1) * sizeof(T));
    if (e == hipSuccess) ptrs.push_back(p);
    *out = (T*)p;
    return e;
  }
};

template <typename T>
hipError_t put(Bufs& b, T** out, const std::vector<T>& v, hipStream_t st) {
  hipError_t e = b.get(out, v.size());
  if (e == hipSuccess && !v.empty())
    e = hipMemcpyAsync(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st);
  return e;
}

// The fronts of a level are launched in groups of at most GROUP fronts, so
// that the per-front scratch of a panel step (Y parts, partial products) is
// sized by a group, not by a level of a large forest.
constexpr size_t GROUP = 16384;

// One launch group: a contiguous range of a level's front list.
struct GroupDev {
  int64_t list_off = 0;  // into the device front lists
  int nf = 0;
  int max_panels = 0;
  int ysplit = 1;        // K parts of the Y product
  int64_t ylev = 0;      // doubles of one K part's Y buffer
  bool whole = true;     // k_finish<true>: one workgroup per front
  int64_t part = 0;      // doubles of the row tiles' partial products (else)
  int64_t maxq = 0;      // largest update set
  std::vector<int> mt;   // per panel: row tiles after it
  std::vector<int> ut;   // per panel: update tiles
  int maxF = 0;          // largest front
};

struct LevelDev {
  int64_t ent_off = 0, ent_n = 0;
  int nf = 0;
  std::vector<GroupDev> groups;
};

reff_status dev_status(hipError_t e, const char* what) {
  return host_fail(e == hipErrorOutOfMemory ? REFF_ERR_OUT_OF_MEMORY : REFF_ERR_DEVICE,
                   std::string(what) + ": " + hipGetErrorString(e));
}

}  // namespace

std::shared_ptr<SelinvPlan> selinv_plan_of(reff_pdn_t* p, reff_status& s) {
  s = REFF_OK;
  if (p->sel_plan) return p->sel_plan;
  auto plan = std::make_shared<SelinvPlan>();
  std::string err;
  if (!build_selinv_plan(p->nt, p->nx, p->ny, p->gx.data(), p->gy.data(),
                         (int32_t)(p->tsv_xy.size() / 2), p->tsv_xy.data(), p->tsv_g.data(),
                         (int32_t)(p->pad_xy.size() / 2), p->pad_xy.data(), LEAF_AREA, *plan,
                         err)) {
    s = host_fail(REFF_ERR_DEVICE, "selected inversion plan: " + err);
    return nullptr;
  }
  p->sel_plan = plan;
  return plan;
}

// Parts the K range of a group's Y products is split into: enough
// workgroups to fill the chip where a group has few fronts, at least 128
// rows of K per part, and at most 1 GiB of partial products.
int group_ysplit(const SelinvPlan& P, const int32_t* fronts, size_t nf, int64_t yb) {
  int64_t tiles0 = 0, maxm = 0;
  for (size_t j = 0; j < nf; ++j) {
    const SnFront& f = P.fronts[(size_t)fronts[j]];
    if (f.k == 0) continue;
    const int64_t m0 = f.F - std::min(PT, f.k);
    tiles0 += (m0 + PT - 1) / PT;
    maxm = std::max(maxm, m0);
  }
  if (tiles0 == 0) return 1;
  int64_t sp = std::min<int64_t>((2048 + tiles0 - 1) / tiles0, 16);
  sp = std::min<int64_t>(sp, std::max<int64_t>(1, maxm / 128));
  while (sp > 1 && sp * yb > ((int64_t)1 << 27)) --sp;
  return (int)std::max<int64_t>(1, sp);
}

// Row tiles after a front's first panel.
int64_t front_tiles(const SnFront& f) {
  return f.k > 0 ? (f.F - std::min(PT, f.k) + PT - 1) / PT : 0;
}

// One workgroup finishes a whole front's panel where a launch has a
// workgroup for every CU that way or the fronts have at most two row tiles (a
// second launch would cost more than the tiles side by side save).
constexpr int WHOLE_FRONTS = 512;
constexpr int WHOLE_TILES = 2;

// The launch groups of every level, with their scratch sizes.
std::vector<std::vector<GroupDev>> plan_groups(const SelinvPlan& P) {
  std::vector<std::vector<GroupDev>> out(P.levels.size());
  for (size_t d = 0; d < P.levels.size(); ++d) {
    const SelinvLevel& L = P.levels[d];
    for (size_t b = 0; b < L.fronts.size(); b += GROUP) {
      GroupDev g;
      g.list_off = (int64_t)b;  // within the level; made absolute by the device build
      g.nf = (int)std::min(GROUP, L.fronts.size() - b);
      for (int j = 0; j < g.nf; ++j) {
        const SnFront& f = P.fronts[(size_t)L.fronts[b + (size_t)j]];
        g.max_panels = std::max(g.max_panels, (f.k + PT - 1) / PT);
        g.ylev += (int64_t)f.F * PT;
        g.part += front_tiles(f) * PT * PT;
        g.maxq = std::max<int64_t>(g.maxq, (int64_t)(f.F - f.k));
        g.maxF = std::max(g.maxF, f.F);
      }
      g.mt.assign((size_t)g.max_panels, 0);
      g.ut.assign((size_t)g.max_panels, 0);
      for (int j = 0; j < g.nf; ++j) {
        const SnFront& f = P.fronts[(size_t)L.fronts[b + (size_t)j]];
        for (int jp = 0; PT * jp < f.k; ++jp) {
          const int m = f.F - PT * jp - std::min(PT, f.k - PT * jp);
          g.mt[(size_t)jp] = std::max(g.mt[(size_t)jp], (m + PT - 1) / PT);
          g.ut[(size_t)jp] = std::max(g.ut[(size_t)jp], update_tiles(f.F, f.k, jp));
        }
      }
      g.ysplit = group_ysplit(P, L.fronts.data() + b, (size_t)g.nf, g.ylev);
      g.whole = g.nf >= WHOLE_FRONTS || g.max_panels == 0 || g.mt[0] <= WHOLE_TILES;
      if (g.whole) g.part = 0;
      out[d].push_back(std::move(g));
    }
  }
  return out;
}

// Scratch sizes of a plan on the device, in doubles / bytes.
struct SelinvSizes {
  int64_t part = 0, ysp = 0;
  int64_t bytes = 0;
};

SelinvSizes selinv_sizes(const SelinvPlan& P) {
  SelinvSizes z;
  for (const auto& lev : plan_groups(P))
    for (const GroupDev& g : lev) {
      z.part = std::max(z.part, g.part);
      if (g.ysplit > 1) z.ysp = std::max(z.ysp, g.ysplit * g.ylev);
    }
  int64_t ent = 0, inv = 0;
  for (const SelinvLevel& L : P.levels) ent += (int64_t)L.ent_idx.size();
  for (const SnFront& f : P.fronts)
    if (f.parent >= 0) inv += P.fronts[(size_t)f.parent].F;
  z.bytes = 8 * (P.arena + z.part + z.ysp + P.n) + 16 * ent +
            (int64_t)sizeof(DFront) * (int64_t)P.fronts.size() + 4 * (inv + (int64_t)P.rel.size()) +
            8 * (int64_t)P.piv_node.size();
  return z;
}

// Device state of a handle's plan: the uploaded tables and every work
// buffer, allocated on the first call and kept with the handle.
// A batch of plans can need 100 GB of fronts, and mapping that much device
// memory afresh costs up to seconds per call; the batch path therefore
// carves its buffers from one workspace per device that is kept between
// calls (grown when a call needs more; reff_release_cached_memory frees
// it).  A call that finds it in use allocates its own.
struct WorkspaceCache {
  std::mutex mu;
  void* p = nullptr;
  size_t bytes = 0;
  bool busy = false;
};
WorkspaceCache g_ws[64];

constexpr size_t ALIGN = 256;
size_t aligned(size_t b) { return (std::max<size_t>(b, 1) + ALIGN - 1) / ALIGN * ALIGN; }

struct SelinvDevice {
  std::vector<LevelDev> lv;
  SelinvSizes sz;
  double *ar = nullptr, *part = nullptr, *Ysp = nullptr, *Rfull = nullptr, *vals = nullptr;
  int64_t *idx = nullptr, *piv = nullptr;
  int32_t *rel = nullptr, *inv = nullptr, *dl = nullptr;
  DFront* dF = nullptr;
  int* bad = nullptr;
  std::vector<void*> ptrs;       // own allocations
  WorkspaceCache* ws = nullptr;  // or buffers carved from a cached workspace
  char* carve = nullptr;
  size_t carve_left = 0;
  ~SelinvDevice() {
    for (void* q : ptrs) (void)hipFree(q);
    if (ws) {
      std::lock_guard<std::mutex> lk(ws->mu);
      ws->busy = false;
    }
  }
  // Take `total` bytes from the device's cached workspace for the buffers
  // that follow (false: use own allocations).
  hipError_t reserve(size_t total, bool& from_cache) {
    from_cache = false;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= 64) return e;
    WorkspaceCache& c = g_ws[dev];
    std::lock_guard<std::mutex> lk(c.mu);
    if (c.busy) return hipSuccess;
    if (c.bytes < total) {
      if (c.p) (void)hipFree(c.p);
      c.p = nullptr;
      c.bytes = 0;
      e = hipMalloc(&c.p, total);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        c.p = nullptr;
        return hipSuccess;  // fall back to own allocations
      }
      c.bytes = total;
    }
    c.busy = true;
    ws = &c;
    carve = (char*)c.p;
    carve_left = c.bytes;
    from_cache = true;
    return hipSuccess;
  }
  template <typename T>
  hipError_t get(T** out, size_t count) {
    const size_t b = aligned(count * sizeof(T));
    if (ws && b <= carve_left) {
      *out = (T*)carve;
      carve += b;
      carve_left -= b;
      return hipSuccess;
    }
    void* q = nullptr;
    ptrs.reserve(ptrs.size() + 1);
    hipError_t e = hipMalloc(&q, b);
    if (e == hipSuccess) ptrs.push_back(q);
    *out = (T*)q;
    return e;
  }
  template <typename T>
  hipError_t put(T** out, const std::vector<T>& v) {
    hipError_t e = get(out, v.size());
    if (e == hipSuccess && !v.empty())
      e = hipMemcpy(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
    return e;
  }
};

std::shared_ptr<SelinvDevice> selinv_device_build(const SelinvPlan& P, reff_status& s,
                                                  bool use_cache = false) {
  s = REFF_OK;
  auto D = std::make_shared<SelinvDevice>();
  std::vector<DFront> dfr(P.fronts.size());
  std::vector<int32_t> lists;
  int64_t n_ent = 0, n_inv = 0;
  D->sz = selinv_sizes(P);
  auto groups = plan_groups(P);
  D->lv.resize(P.levels.size());
  for (size_t d = 0; d < P.levels.size(); ++d) {
    const SelinvLevel& L = P.levels[d];
    LevelDev& V = D->lv[d];
    V.nf = (int)L.fronts.size();
    V.ent_off = n_ent;
    V.ent_n = (int64_t)L.ent_idx.size();
    n_ent += V.ent_n;
    const int64_t lbase = (int64_t)lists.size();
    for (GroupDev& g : groups[d]) {
      int64_t yb = 0, pa = 0;
      for (int j = 0; j < g.nf; ++j) {
        const int32_t i = L.fronts[(size_t)(g.list_off + j)];
        const SnFront& f = P.fronts[(size_t)i];
        DFront& x = dfr[(size_t)i];
        x.off = f.off;
        x.poff = f.parent >= 0 ? P.fronts[(size_t)f.parent].off : -1;
        x.rel = f.rel;
        x.piv = f.piv;
        x.F = f.F;
        x.k = f.k;
        x.child[0] = x.child[1] = -1;
        x.pF = f.parent >= 0 ? P.fronts[(size_t)f.parent].F : 0;
        x.inv = n_inv;
        n_inv += x.pF;
        x.ybuf = yb;
        x.part = pa;
        yb += (int64_t)f.F * PT;
        pa += front_tiles(f) * PT * PT;
      }
      g.list_off += lbase;
    }
    lists.insert(lists.end(), L.fronts.begin(), L.fronts.end());
    V.groups = std::move(groups[d]);
  }
  for (size_t i = 0; i < P.fronts.size(); ++i)
    if (has_update(P.fronts[i])) dfr[(size_t)P.fronts[i].parent].child[P.fronts[i].rank] = (int32_t)i;
  hipError_t e = hipSuccess;
  if (use_cache) {
    const SelinvSizes& z = D->sz;
    const size_t total = aligned(8 * (size_t)P.arena) + aligned(8 * (size_t)z.part) +
                         aligned(8 * (size_t)z.ysp) + aligned(8 * (size_t)P.n) + aligned(4) +
                         2 * aligned(8 * (size_t)n_ent) + aligned(8 * P.piv_node.size()) +
                         aligned(4 * P.rel.size()) + aligned(4 * (size_t)n_inv) + aligned(4 * lists.size()) +
                         aligned(sizeof(DFront) * dfr.size());
    bool cached = false;
    e = D->reserve(total, cached);
  }
  if (e == hipSuccess) e = D->get(&D->ar, (size_t)P.arena);
  if (e == hipSuccess) e = D->get(&D->part, (size_t)D->sz.part);
  if (e == hipSuccess) e = D->get(&D->Ysp, (size_t)D->sz.ysp);
  if (e == hipSuccess) e = D->get(&D->Rfull, (size_t)P.n);
  if (e == hipSuccess) e = D->get(&D->bad, 1);
  // G's entries, level by level straight from the plan
  if (e == hipSuccess) e = D->get(&D->idx, (size_t)n_ent);
  if (e == hipSuccess) e = D->get(&D->vals, (size_t)n_ent);
  for (size_t d = 0; d < P.levels.size() && e == hipSuccess; ++d) {
    const SelinvLevel& L = P.levels[d];
    const LevelDev& V = D->lv[d];
    if (V.ent_n == 0) continue;
    e = hipMemcpy(D->idx + V.ent_off, L.ent_idx.data(), sizeof(int64_t) * V.ent_n,
                  hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = hipMemcpy(D->vals + V.ent_off, L.ent_val.data(), sizeof(double) * V.ent_n,
                    hipMemcpyHostToDevice);
  }
  if (e == hipSuccess) e = D->put(&D->piv, P.piv_node);
  if (e == hipSuccess) e = D->put(&D->rel, P.rel);
  if (e == hipSuccess) e = D->put(&D->dl, lists);
  if (e == hipSuccess) e = D->put(&D->dF, dfr);
  if (e == hipSuccess) e = D->get(&D->inv, (size_t)n_inv);
  if (e == hipSuccess && !dfr.empty()) {
    hipLaunchKernelGGL(k_invert_rel, dim3((unsigned)std::min<size_t>(dfr.size(), 65536)), dim3(256),
                       0, nullptr, (const DFront*)D->dF, (int)dfr.size(), (const int32_t*)D->rel,
                       D->inv);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  }
  if (e != hipSuccess) {
    s = dev_status(e, "selected inversion: allocation / upload");
    return nullptr;
  }
  return D;
}

std::shared_ptr<SelinvDevice> selinv_device_of(reff_pdn_t* p, const SelinvPlan& P,
                                               reff_status& s) {
  s = REFF_OK;
  if (p->sel_dev) return p->sel_dev;
  auto D = selinv_device_build(P, s);
  if (D) p->sel_dev = D;
  return D;
}

// The numeric work of a plan on its device state, on `st`: factorisation
// (deepest level first) then selected inversion (roots first); D.Rfull
// receives R for every pivot node (0 elsewhere).  t_fact: when the
// factorisation finished (the call synchronises there to read the pivot
// flag).
reff_status selinv_run(const SelinvPlan& P, const SelinvDevice& D, hipStream_t st_,
                       std::chrono::steady_clock::time_point& t_fact,
                       const std::vector<uint8_t>* need = nullptr) {
  double *ar = D.ar, *part = D.part, *Ysp = D.Ysp;
  double* Rfull = D.Rfull;
  const int32_t *rel = D.rel, *dl = D.dl;
  const DFront* dF = D.dF;
  int* bad = D.bad;
  hipLaunchKernelGGL(k_zero, flat(P.n), dim3(256), 0, st_, Rfull, P.n);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemsetAsync(bad, 0, sizeof(int), st_);
  auto gy = [](int nf) { return (unsigned)std::min<int64_t>(nf, MAX_GY); };
  const int nlev = (int)P.levels.size();
  // factorisation, deepest level first
  for (int d = nlev - 1; d >= 0 && e == hipSuccess; --d) {
    const LevelDev& V = D.lv[(size_t)d];
    if (V.nf == 0) continue;
    for (const GroupDev& G : V.groups)
      if (G.maxF > 0)
        hipLaunchKernelGGL(k_assemble, dim3((unsigned)((G.maxF + 4 * AC - 1) / (4 * AC)), gy(G.nf)),
                           dim3(256), 0, st_, dF, dl + G.list_off, G.nf, (const int32_t*)D.inv, ar);
    if (V.ent_n > 0)
      hipLaunchKernelGGL(k_scatter_add, flat(V.ent_n), dim3(256), 0, st_, D.idx + V.ent_off,
                         D.vals + V.ent_off, V.ent_n, ar);
    for (const GroupDev& G : V.groups) {
      const int32_t* l = dl + G.list_off;
      for (int jp = 0; jp < G.max_panels; ++jp) {
        hipLaunchKernelGGL(k_tile, dim3(gy(G.nf)), dim3(256), 0, st_, dF, l, G.nf, jp, ar, bad);
        const int mt = G.mt[(size_t)jp];
        if (mt == 0) continue;
        hipLaunchKernelGGL(k_front_gemm<OP_LHAT>, dim3((unsigned)mt, gy(G.nf)), dim3(256), 0,
                           st_, dF, l, G.nf, jp, ar, mt, 1, Ysp, (int64_t)0);
        hipLaunchKernelGGL(k_front_gemm<OP_UPDATE>, dim3((unsigned)G.ut[(size_t)jp], gy(G.nf)),
                           dim3(256), 0, st_, dF, l, G.nf, jp, ar, mt, 1, Ysp, (int64_t)0);
      }
    }
    e = hipGetLastError();
  }
  int hbad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st_);
  if (e == hipSuccess) e = hipStreamSynchronize(st_);
  if (e != hipSuccess) return dev_status(e, "selected inversion: factorisation");
  if (hbad) return host_fail(REFF_ERR_DEVICE, "sparse factorisation: a pivot was not positive");
  t_fact = std::chrono::steady_clock::now();
  // With a request, the selected inversion visits only the needed fronts:
  // each launch group runs over the compacted list of its needed fronts
  // (their scratch slots and Y offsets are those of the full group).
  Bufs lb;
  int32_t* dact = nullptr;
  std::vector<std::vector<std::pair<int64_t, int>>> act_rng(P.levels.size());
  if (need) {
    std::vector<int32_t> act;
    for (size_t d = 0; d < P.levels.size(); ++d) {
      const SelinvLevel& L = P.levels[d];
      for (const GroupDev& G : D.lv[d].groups) {
        const int64_t lbase = G.list_off - D.lv[d].groups.front().list_off;
        const int64_t a0 = (int64_t)act.size();
        for (int j = 0; j < G.nf; ++j) {
          const int32_t fi = L.fronts[(size_t)(lbase + j)];
          if ((*need)[(size_t)fi]) act.push_back(fi);
        }
        act_rng[d].push_back({a0, (int)((int64_t)act.size() - a0)});
      }
    }
    e = put(lb, &dact, act, st_);
    if (e == hipSuccess) e = hipStreamSynchronize(st_);
    if (e != hipSuccess) return dev_status(e, "selected inversion: request lists");
  }
  // selected inversion, roots first
  for (int d = 0; d < nlev && e == hipSuccess; ++d) {
    const LevelDev& V = D.lv[(size_t)d];
    for (size_t gi = 0; gi < V.groups.size(); ++gi) {
      const GroupDev& G = V.groups[gi];
      const int32_t* l = dl + G.list_off;
      int nfa = G.nf;
      if (need) {
        l = dact + act_rng[(size_t)d][gi].first;
        nfa = act_rng[(size_t)d][gi].second;
        if (nfa == 0) continue;
      }
      if (d > 0 && G.maxq > 0) {
        const unsigned gx = (unsigned)std::max<int64_t>(1, (G.maxq + 3) / 4);
        hipLaunchKernelGGL(k_gather, dim3(gx, gy(nfa)), dim3(256), 0, st_, dF, l, nfa, rel, ar);
      }
      for (int jp = G.max_panels - 1; jp >= 0; --jp) {
        const int mt = G.mt[(size_t)jp];
        if (mt > 0)
          hipLaunchKernelGGL(k_front_gemm<OP_Y>, dim3((unsigned)(mt * G.ysplit), gy(nfa)),
                             dim3(256), 0, st_, dF, l, nfa, jp, ar, mt, G.ysplit, Ysp, G.ylev);
        if (G.whole) {
          hipLaunchKernelGGL(k_finish<true>, dim3(1, gy(nfa)), dim3(256), 0, st_, dF, l, nfa, jp, ar,
                             G.ysplit, (const double*)Ysp, G.ylev, part, D.piv, Rfull);
        } else {
          if (mt > 0)
            hipLaunchKernelGGL(k_finish<false>, dim3((unsigned)mt, gy(nfa)), dim3(256), 0, st_, dF,
                               l, nfa, jp, ar, G.ysplit, (const double*)Ysp, G.ylev, part, D.piv,
                               Rfull);
          hipLaunchKernelGGL(k_zpp, dim3(4, gy(nfa)), dim3(256), 0, st_, dF, l, nfa, jp, ar,
                             (const double*)part, D.piv, Rfull);
        }
      }
    }
    e = hipGetLastError();
  }
  if (e != hipSuccess) return dev_status(e, "selected inversion");
  return REFF_OK;
}

}  // namespace reff

extern "C" {

reff_status reff_selinv_info(const reff_pdn_desc* d, reff_selinv_stats* info) try {
  using namespace reff;
  if (!d || !info) return host_fail(REFF_ERR_INVALID_ARG, "NULL descriptor or info");
  reff_status s = host_validate_desc(d);
  if (s != REFF_OK) return s;
  SelinvPlan plan;
  std::string err;
  bool dis = false;
  if (!build_selinv_plan(d->n_tiers, d->nx, d->ny, d->gx, d->gy, d->n_tsv, d->tsv_xy, d->tsv_g,
                         d->n_pads, d->pad_xy, LEAF_AREA, plan, err, &dis))
    return host_fail(dis ? REFF_ERR_DISCONNECTED : REFF_ERR_INVALID_ARG,
                     "selected inversion plan: " + err);
  std::memset(info, 0, sizeof(*info));
  info->n_fronts = (int64_t)plan.fronts.size();
  info->n_levels = (int32_t)plan.levels.size();
  for (const SnFront& f : plan.fronts) info->max_front = std::max<int64_t>(info->max_front, f.F);
  info->device_bytes = selinv_sizes(plan).bytes;
  info->flops_factor = plan.flops_factor;
  info->flops_selinv = plan.flops_selinv;
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}

reff_status reff_selinv_diag(reff_pdn p, const int64_t* nodes, int64_t n_nodes, double* R_out,
                             const reff_solve_opts* opts, reff_selinv_stats* st) try {
  using namespace reff;
  const auto t0 = std::chrono::steady_clock::now();
  if (!p) return host_fail(REFF_ERR_INVALID_ARG, "handle is NULL");
  if (nodes && n_nodes < 0) return host_fail(REFF_ERR_INVALID_ARG, "n_nodes < 0");
  const int64_t count = nodes ? n_nodes : p->n;
  if (count > 0 && !R_out) return host_fail(REFF_ERR_INVALID_ARG, "R_out is NULL");
  for (int64_t i = 0; nodes && i < count; ++i)
    if (nodes[i] < 0 || nodes[i] >= p->n)
      return host_fail(REFF_ERR_INVALID_ARG, "node id " + std::to_string(nodes[i]) + " out of range");
  hipStream_t st_ = opts ? (hipStream_t)opts->stream : nullptr;
  const bool out_dev = opts && opts->out_on_device;
  if (opts && opts->out_on_device != 0 && opts->out_on_device != 1)
    return host_fail(REFF_ERR_INVALID_ARG, "out_on_device must be 0 or 1");
  hipError_t e = hipSetDevice(p->device);
  if (e != hipSuccess) return dev_status(e, "hipSetDevice");
  reff_status s;
  auto plan_sp = selinv_plan_of(p, s);
  if (!plan_sp) return s;
  const SelinvPlan& P = *plan_sp;
  const auto t_plan = std::chrono::steady_clock::now();

  auto dev_sp = selinv_device_of(p, P, s);
  if (!dev_sp) return s;
  const SelinvDevice& D = *dev_sp;
  const auto t_setup = std::chrono::steady_clock::now();
  double* Rfull = D.Rfull;
  Bufs b;
  double* dout = nullptr;
  int64_t* dnodes = nullptr;
  if (nodes && count > 0) {
    std::vector<int64_t> nv(nodes, nodes + count);
    e = put(b, &dnodes, nv, st_);
    // the staged host vector must outlive the copy
    if (e == hipSuccess) e = hipStreamSynchronize(st_);
  }
  if (e == hipSuccess && !out_dev && count > 0) e = b.get(&dout, (size_t)count);
  if (e != hipSuccess) return dev_status(e, "selected inversion: output buffers");
  // a node list needs only its fronts and their ancestors inverted
  double fl_sel = P.flops_selinv;
  std::vector<uint8_t> need;
  if (nodes) need = needed_fronts(P, std::vector<int64_t>(nodes, nodes + count), &fl_sel);
  std::chrono::steady_clock::time_point t_fact;
  s = selinv_run(P, D, st_, t_fact, nodes ? &need : nullptr);
  if (s != REFF_OK) return s;
  // output
  if (e == hipSuccess && count > 0) {
    double* out = out_dev ? R_out : dout;
    if (nodes) {
      hipLaunchKernelGGL(k_pick, flat(count), dim3(256), 0, st_, Rfull, dnodes, count, out);
      e = hipGetLastError();
    } else {
      e = hipMemcpyAsync(out, Rfull, sizeof(double) * count, hipMemcpyDeviceToDevice, st_);
    }
    if (e == hipSuccess && !out_dev)
      e = hipMemcpyAsync(R_out, dout, sizeof(double) * count, hipMemcpyDeviceToHost, st_);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st_);
  if (e != hipSuccess) return dev_status(e, "selected inversion");
  const auto t1 = std::chrono::steady_clock::now();
  if (st) {
    std::memset(st, 0, sizeof(*st));
    st->n_fronts = (int64_t)P.fronts.size();
    st->n_levels = (int32_t)P.levels.size();
    for (const SnFront& f : P.fronts) st->max_front = std::max<int64_t>(st->max_front, f.F);
    st->device_bytes = D.sz.bytes;
    st->flops_factor = P.flops_factor;
    st->flops_selinv = fl_sel;
    st->seconds = std::chrono::duration<double>(t1 - t0).count();
    st->seconds_plan = std::chrono::duration<double>(t_plan - t0).count();
    st->seconds_factor = std::chrono::duration<double>(t_fact - t_plan).count();
    st->seconds_selinv = std::chrono::duration<double>(t1 - t_fact).count();
    st->seconds_setup = std::chrono::duration<double>(t_setup - t_plan).count();
  }
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}

reff_status reff_release_cached_memory(int32_t device) try {
  using namespace reff;
  if (device < 0 || device >= 64) return host_fail(REFF_ERR_INVALID_ARG, "bad device");
  WorkspaceCache& c = g_ws[device];
  std::lock_guard<std::mutex> lk(c.mu);
  if (!c.p || c.busy) return REFF_OK;
  hipError_t e = hipSetDevice(device);
  if (e == hipSuccess) e = hipFree(c.p);
  c.p = nullptr;
  c.bytes = 0;
  if (e != hipSuccess) return dev_status(e, "releasing cached memory");
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}

reff_status reff_selinv_batch(const reff_pdn_desc* plans, int32_t n_plans,
                              const int64_t* const* nodes, const int64_t* n_nodes,
                              double* const* R_out, const reff_solve_opts* opts,
                              reff_selinv_stats* st) try {
  using namespace reff;
  const auto t0 = std::chrono::steady_clock::now();
  if (st) std::memset(st, 0, sizeof(*st));
  if (n_plans < 0) return host_fail(REFF_ERR_INVALID_ARG, "n_plans < 0");
  if (n_plans == 0) return REFF_OK;
  if (!plans || !R_out) return host_fail(REFF_ERR_INVALID_ARG, "NULL plans or R_out");
  if (opts && opts->out_on_device != 0 && opts->out_on_device != 1)
    return host_fail(REFF_ERR_INVALID_ARG, "out_on_device must be 0 or 1");
  const bool out_dev = opts && opts->out_on_device;
  hipStream_t st_ = opts ? (hipStream_t)opts->stream : nullptr;
  const size_t np = (size_t)n_plans;
  std::vector<int64_t> cnt(np);
  // descriptors checked on host threads; the first bad plan is reported
  std::vector<reff_status> vs(np, REFF_OK);
  std::vector<std::string> vm(np);
  selinv_parallel_for(np, [&](size_t i) {
    vs[i] = host_validate_desc(&plans[i]);
    if (vs[i] != REFF_OK) vm[i] = reff_last_error();  // this thread's message
  });
  for (size_t i = 0; i < np; ++i) {
    const std::string who = "plan " + std::to_string(i) + ": ";
    if (vs[i] != REFF_OK) return host_fail(vs[i], who + vm[i]);
    const int64_t n = (int64_t)plans[i].n_tiers * plans[i].nx * plans[i].ny;
    const bool given = nodes && nodes[i];
    if (given && (!n_nodes || n_nodes[i] < 0)) return host_fail(REFF_ERR_INVALID_ARG, who + "bad n_nodes");
    cnt[i] = given ? n_nodes[i] : n;
    if (cnt[i] > 0 && !R_out[i]) return host_fail(REFF_ERR_INVALID_ARG, who + "R_out NULL");
    for (int64_t k = 0; given && k < cnt[i]; ++k)
      if (nodes[i][k] < 0 || nodes[i][k] >= n)
        return host_fail(REFF_ERR_INVALID_ARG,
                         who + "node id " + std::to_string(nodes[i][k]) + " out of range");
  }
  // Plans are taken in chunks of consecutive plans with about equal node
  // counts (one chunk below 4M nodes, at most four): the host analysis of
  // chunk c + 1 runs on host threads while the device factors and inverts
  // chunk c, and each chunk is one forest (the plans' trees merged by
  // depth) on the device workspace.
  int64_t tot_n = 0;
  std::vector<int64_t> pn(np);
  for (size_t i = 0; i < np; ++i) {
    pn[i] = (int64_t)plans[i].n_tiers * plans[i].nx * plans[i].ny;
    tot_n += pn[i];
  }
  const int64_t nch = std::max<int64_t>(
      1, std::min<int64_t>({(int64_t)4, (int64_t)np, tot_n / (int64_t(4) << 20)}));
  std::vector<size_t> cb{0};
  {
    const int64_t share = (tot_n + nch - 1) / nch;
    int64_t acc = 0;
    for (size_t i = 0; i < np; ++i) {
      acc += pn[i];
      if (acc >= share * (int64_t)cb.size() && (int64_t)cb.size() < nch && i + 1 < np)
        cb.push_back(i + 1);
    }
    cb.push_back(np);
  }
  struct Chunk {
    SelinvPlan P;
    std::vector<int64_t> base;
    reff_status s = REFF_OK;
    std::string err;
  };
  auto analyse = [&](size_t c, Chunk& out) {
    const size_t p0 = cb[c], p1 = cb[c + 1];
    std::vector<SelinvPlan> sp(p1 - p0);
    std::vector<std::string> err(p1 - p0);
    std::vector<char> ok(p1 - p0, 0), disc(p1 - p0, 0);
    selinv_parallel_for(p1 - p0, [&](size_t k) {
      const reff_pdn_desc& d = plans[p0 + k];
      bool dis = false;
      ok[k] = build_selinv_plan(d.n_tiers, d.nx, d.ny, d.gx, d.gy, d.n_tsv, d.tsv_xy, d.tsv_g,
                                d.n_pads, d.pad_xy, LEAF_AREA, sp[k], err[k], &dis);
      disc[k] = dis;
    });
    for (size_t k = 0; k < p1 - p0; ++k)
      if (!ok[k]) {
        out.s = disc[k] ? REFF_ERR_DISCONNECTED : REFF_ERR_INVALID_ARG;
        out.err = "plan " + std::to_string(p0 + k) + ": " + err[k];
        return;
      }
    out.P = merge_selinv_plans(sp, out.base);
  };
  // the same on a thread of its own, which must not throw
  auto analyse_ahead = [&](size_t c, Chunk& out) {
    try {
      analyse(c, out);
    } catch (...) {
      out.s = host_exception();  // (its text stays with this thread)
      out.err.clear();
    }
  };
  // requested nodes of every plan, in plan order, into one device array
  int64_t total = 0;
  std::vector<int64_t> out_at(np + 1, 0);
  for (size_t i = 0; i < np; ++i) out_at[i + 1] = out_at[i] + cnt[i];
  total = out_at[np];
  double t_plan = 0.0, t_setup = 0.0, t_factor = 0.0, t_selinv = 0.0;
  int64_t n_fronts = 0, max_front = 0, dev_bytes = 0;
  int32_t n_levels = 0;
  double fl_fact = 0.0, fl_sel = 0.0;
  auto tp = std::chrono::steady_clock::now();
  auto cur = std::make_unique<Chunk>();
  analyse(0, *cur);
  t_plan += std::chrono::duration<double>(std::chrono::steady_clock::now() - tp).count();
  // a plan of the first chunk that fails its analysis is refused before any
  // device work; later chunks' failures come after earlier chunks' device
  // work, with nothing written to R_out either way
  if (cur->s != REFF_OK) return host_fail(cur->s, cur->err);
  Bufs b;
  double* dres = nullptr;
  hipError_t e = b.get(&dres, (size_t)total);
  if (e != hipSuccess) return dev_status(e, "selected inversion batch: output");
  for (size_t c = 0; c + 1 < cb.size(); ++c) {
    if (cur->s != REFF_OK)
      return host_fail(cur->s, cur->err.empty() ? "analysis of a later chunk of plans" : cur->err);
    auto next = std::make_unique<Chunk>();
    std::thread ahead;
    if (c + 2 < cb.size()) {
      try {
        ahead = std::thread([&, c] { analyse_ahead(c + 1, *next); });
      } catch (const std::system_error&) {  // no thread to be had: analysed below
      }
    }
    struct Join {
      std::thread& t;
      ~Join() {
        if (t.joinable()) t.join();
      }
    } join{ahead};
    const SelinvPlan& P = cur->P;
    const size_t p0 = cb[c], p1 = cb[c + 1];
    const auto t0c = std::chrono::steady_clock::now();
    reff_status s;
    auto dev_sp = selinv_device_build(P, s, true);
    if (!dev_sp) return s;
    const SelinvDevice& D = *dev_sp;
    const auto t_set = std::chrono::steady_clock::now();
    std::vector<int64_t> ids;
    ids.reserve((size_t)(out_at[p1] - out_at[p0]));
    bool every = true;
    for (size_t i = p0; i < p1; ++i) {
      const bool given = nodes && nodes[i];
      every = every && !given;
      for (int64_t k = 0; k < cnt[i]; ++k)
        ids.push_back(cur->base[i - p0] + (given ? nodes[i][k] : k));
    }
    // with node lists, only their fronts and ancestors are inverted
    double fl = P.flops_selinv;
    std::vector<uint8_t> need;
    if (!every) need = needed_fronts(P, ids, &fl);
    std::chrono::steady_clock::time_point t_fact;
    s = selinv_run(P, D, st_, t_fact, every ? nullptr : &need);
    if (s != REFF_OK) return s;
    Bufs bc;
    int64_t* dids = nullptr;
    e = put(bc, &dids, ids, st_);
    const int64_t nc = (int64_t)ids.size();
    if (e == hipSuccess && nc > 0) {
      hipLaunchKernelGGL(k_pick, flat(nc), dim3(256), 0, st_, D.Rfull, dids, nc,
                         dres + out_at[p0]);
      e = hipGetLastError();
    }
    // the workspace and the staged ids are reused or freed after this
    if (e == hipSuccess) e = hipStreamSynchronize(st_);
    if (e != hipSuccess) return dev_status(e, "selected inversion batch");
    const auto t_end = std::chrono::steady_clock::now();
    t_setup += std::chrono::duration<double>(t_set - t0c).count();
    t_factor += std::chrono::duration<double>(t_fact - t_set).count();
    t_selinv += std::chrono::duration<double>(t_end - t_fact).count();
    n_fronts += (int64_t)P.fronts.size();
    n_levels = std::max<int32_t>(n_levels, (int32_t)P.levels.size());
    for (const SnFront& f : P.fronts) max_front = std::max<int64_t>(max_front, f.F);
    dev_bytes = std::max<int64_t>(dev_bytes, D.sz.bytes);
    fl_fact += P.flops_factor;
    fl_sel += fl;
    dev_sp.reset();
    // the next chunk's analysis: whatever of it the device work did not hide
    const auto tw = std::chrono::steady_clock::now();
    if (ahead.joinable())
      ahead.join();
    else if (c + 2 < cb.size())
      analyse(c + 1, *next);
    t_plan += std::chrono::duration<double>(std::chrono::steady_clock::now() - tw).count();
    cur = std::move(next);
  }
  std::vector<double> host;
  if (!out_dev) {
    host.resize((size_t)total);
    if (total > 0)
      e = hipMemcpyAsync(host.data(), dres, sizeof(double) * total, hipMemcpyDeviceToHost, st_);
  }
  for (size_t i = 0; i < np && e == hipSuccess; ++i)
    if (cnt[i] > 0 && out_dev)
      e = hipMemcpyAsync(R_out[i], dres + out_at[i], sizeof(double) * cnt[i],
                         hipMemcpyDeviceToDevice, st_);
  if (e == hipSuccess) e = hipStreamSynchronize(st_);
  if (e != hipSuccess) return dev_status(e, "selected inversion batch");
  if (!out_dev)
    for (size_t i = 0; i < np; ++i)
      if (cnt[i] > 0) std::memcpy(R_out[i], host.data() + out_at[i], sizeof(double) * cnt[i]);
  const auto t1 = std::chrono::steady_clock::now();
  if (st) {
    st->n_fronts = n_fronts;
    st->n_levels = n_levels;
    st->max_front = max_front;
    st->device_bytes = dev_bytes;
    st->flops_factor = fl_fact;
    st->flops_selinv = fl_sel;
    st->seconds = std::chrono::duration<double>(t1 - t0).count();
    st->seconds_plan = t_plan;
    st->seconds_setup = t_setup;
    st->seconds_factor = t_factor + t_setup;
    st->seconds_selinv = t_selinv;
  }
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}

}  // extern "C"
