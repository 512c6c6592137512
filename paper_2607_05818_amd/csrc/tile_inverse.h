// Elimination of one 64 x 64 symmetric positive definite tile by a workgroup of
// four waves: the plain inverse (sparse-direct fronts, whose M-matrices lose
// nothing in it), and a guarded symmetric sweep (block solver, reduced pair
// system).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace reff {

constexpr int TILE = 64;

typedef double tile_d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// 1/x and 1/sqrt(x) for x > 0 from the hardware estimates plus two Newton
// steps each (full float64 accuracy, without the long IEEE division and
// square-root sequences, which dominate a latency-bound sweep step).
__device__ __forceinline__ double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ double rsqrt64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * fma(-0.5 * x, y * y, 1.5);
  return y * fma(-0.5 * x, y * y, 1.5);
}

// Inverse of the symmetric positive definite w x w matrix in T (64 x 64 in
// LDS, identity-padded past w), in place, by Gauss-Jordan elimination in four
// blocks of 16 columns; a pivot that is not positive sets *bad.
//
// One wave eliminates a block's 16 columns on all 64 rows in registers (lane
// r holds row r): the pivot row's entries are broadcast by v_readlane, so the
// 16 dependent steps need neither LDS nor barriers.  That leaves the block
// D = A_bb^-1 on its own rows and C = -A_ib D on the others, and the other
// columns follow as one product on the matrix cores, A_ij += C_ib A_bj (and
// A_bj = D A_bj), a 16-row strip per wave.
// The tile's 64 steps are a serial chain, and every panel of every level
// waits for one (98 panels at 4 x 512 x 512): a step costs about 36
// independent register instructions here, against a barrier, LDS reads, a
// square root and a division when the four waves shared each column.  Per
// panel of the root of the 4 x 512 x 512 stack: 20 us, where Cholesky and the
// triangular inverse took 101 us and their repetition in the inversion 60 us.
// The tile is all the LDS it takes (33 KB: four workgroups per CU).
__device__ __forceinline__ void invert_tile(double (*T)[TILE + 1], int w, int* bad) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int cc = lane & 15, kr = lane >> 4;
  for (int b = 0; 16 * b < w; ++b) {
    if (wv == 0) {
      double a[16], own = 1.0;
#pragma unroll
      for (int c = 0; c < 16; ++c) a[c] = T[lane][16 * b + c];
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const int q = 16 * b + p;  // pivot row and column
        const double inv = rcp64(lane_value(a[p], q));
        // row r loses (a_rp inv) * row q; row q is to be multiplied by inv,
        // which waits for the end of the block (own): its later steps are
        // linear in it, and no row reads it again
        own = lane == q ? inv : own;
        const double mult = lane == q ? 0.0 : -a[p] * inv;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          if (c == p) continue;
          a[c] = fma(mult, lane_value(a[c], q), a[c]);
        }
        a[p] = lane == q ? 1.0 : mult;
      }
      if (!(own > 0.0 && std::isfinite(own))) atomicOr(bad, 1);
#pragma unroll
      for (int c = 0; c < 16; ++c) T[lane][16 * b + c] = a[c] * own;
    }
    __syncthreads();
    tile_d4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j == b) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        acc[j][r] = wv == b ? 0.0 : T[16 * wv + kr + 4 * r][16 * j + cc];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(T[16 * wv + cc][16 * b + 4 * ks + kr],
                                                      T[16 * b + 4 * ks + kr][16 * j + cc], acc[j],
                                                      0, 0, 0);
    }
    __syncthreads();  // every strip has read row block b
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j == b) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) T[16 * wv + kr + 4 * r][16 * j + cc] = acc[j][r];
    }
    __syncthreads();
  }
}

// Columns of a block at their sweep steps, times 1/sqrt(pivot).
struct SweepBlock {
  double col[TILE][17];
};

// Guarded symmetric sweep of the Jacobi-scaled matrix in M (LDS), index by
// index in order.  Index j is swept only if its current pivot (the Schur
// complement with respect to the indices swept before it) is above eps;
// otherwise it is dropped as numerically dependent (drop[j]).  Afterwards M
// holds -(A_KK)^-1 on the kept set K.  With WITH_T, column j of the upper
// triangular T = Sc (e_j - beta)/sqrt(pivot) is written to Tl (beta: the
// coefficients of j on the kept earlier indices), so that T^T M T = I on K
// and T has zero columns for dropped j.
//
// Four blocks of 16 columns: one wave sweeps a block on all 64 rows in
// registers (lane r holds row r, the pivot row broadcast by v_readlane: no LDS
// and no barrier in the 16 dependent steps), the others follow as one
// matrix-core product, a 16-row strip per wave.  That product takes each
// step's column as it stood at its step, scaled on both sides alike, A_ij -=
// sum_p u_p(i) u_p(j), and the block's rows are copies of its columns: the
// matrix stays symmetric to the last bit between blocks, and a Schur
// complement is off by roundings of A only.  Near-dependent blocks need that:
// with 64 neighbouring columns and precond_degree 1, the finished inverse of
// the block as a factor, or multipliers against unscaled columns, took two to
// three times the iterations.
// A serial chain of 64 steps that every iteration waits for twice: with a
// barrier and LDS broadcasts per step k_small1 and k_small3 took 48 and 40 us
// on 2 x 32 x 32 nodes, now 36 and 30 (k_small2, products only: 9 and 6).
template <bool WITH_T>
__device__ void sweep_blocks(double (*M)[TILE + 1], SweepBlock& sb, double eps, int* drop,
                             const double* sc, double (*Tl)[TILE + 1]) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cc = lane & 15, kr = lane >> 4;
  uint64_t kept = 0;  // wave 0: swept indices
  // Pivots only fall: a block without one above eps at the start is dropped
  // whole (a solve block of 16 columns takes a quarter of the steps).  Every
  // wave decides from the untouched diagonal, so all take the same barriers.
  const uint64_t live = __ballot(M[lane][lane] > eps);
  __syncthreads();
#pragma unroll 1
  for (int b = 0; b < 4; ++b) {
    if (((live >> (16 * b)) & 0xffff) == 0) {
      if (wv == 0) {
        if (lane < 16) drop[16 * b + lane] = 1;
        if (WITH_T)
#pragma unroll
          for (int p = 0; p < 16; ++p) Tl[lane][16 * b + p] = 0.0;
      }
      continue;
    }
    if (wv == 0) {
      double a[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) a[c] = M[lane][16 * b + c];
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const int q = 16 * b + p;
        const double piv = lane_value(a[p], q);
        const bool dj = !(piv > eps);
        const double rs = rsqrt64(piv), inv = rcp64(piv);
        // a dropped column changes nothing else (no branch: the steps' chains
        // overlap, 40 -> 36 us)
        const double u = dj ? 0.0 : a[p] * rs, f = dj ? 0.0 : a[p] * inv;
        sb.col[lane][p] = u;
        if (WITH_T) {
          const double t = lane < q ? ((kept >> lane) & 1 ? -u : 0.0) : (lane == q && !dj ? rs : 0.0);
          Tl[lane][q] = sc[lane] * t;
        }
        if (lane == 0) drop[q] = dj ? 1 : 0;
        kept |= (uint64_t)(dj ? 0 : 1) << q;
        // row q becomes inv row q, as row q + (inv - 1) row q: pivots of the
        // scaled matrix are at most 1 up to rounding, so nothing cancels
        const double mult = dj ? 0.0 : lane == q ? inv - 1.0 : -f;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          if (c == p) continue;
          a[c] = fma(mult, lane_value(a[c], q), a[c]);
        }
        a[p] = dj ? a[p] : lane == q ? -inv : f;
      }
#pragma unroll
      for (int c = 0; c < 16; ++c) M[lane][16 * b + c] = a[c];
    }
    __syncthreads();
    // rows of the block are its columns; the other strips take the product
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j == b) continue;
      tile_d4 acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * wv + kr + 4 * r;
        acc[r] = wv == b ? M[16 * j + cc][i] : M[i][16 * j + cc];
      }
      if (wv != b) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-sb.col[16 * wv + cc][4 * ks + kr],
                                                     sb.col[16 * j + cc][4 * ks + kr], acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) M[16 * wv + kr + 4 * r][16 * j + cc] = acc[r];
    }
    __syncthreads();
  }
  __syncthreads();  // drop and Tl of blocks dropped whole
}

}  // namespace reff
