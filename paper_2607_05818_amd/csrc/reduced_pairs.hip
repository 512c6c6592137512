// Bump-to-load pair resistances of a stack of uniformly meshed tiers by the
// paper's divide-and-conquer method (Sec. III-C, III-D):
//
//  1. intra-die resistances from the closed form of Eq. 3: TSV-TSV on every
//     tier (d x p x p), bump-TSV on tier 0 (m x p), load-TSV on the last
//     tier (n x p) -- rectangles of one cosine table per tier (grid_pairs.hip);
//  2. the reduced saddle-point system C x = b of size (p+1)(d-1): unknowns
//     are the p TSV currents of each of the d-1 tier interfaces and the d-1
//     supply-voltage differences.  With Atilde^i = -R^i_TT / 2 (TSV-TSV
//     resistances of tier i) the TSV block H is block tridiagonal: diagonal
//     block of interface a = Atilde^a + Atilde^{a+1} + diag(Rt_{., a}),
//     off-diagonal block between interfaces a and a+1 = -Atilde^{a+1}; the
//     constraint block B holds one row of ones per interface (each
//     interface carries the unit current);
//  3. C depends on neither bump nor load, so it is factorised once; each
//     bump i contributes b^1_i = [-R^1_{s_i,.}/2 in interface 0; 1_{d-1}/2]
//     and each load j b^d_j = [-R^d_{s_j,.}/2 in interface d-2; 1_{d-1}/2],
//     so that m + n solves give x^1_i, x^d_j (linearity of Sec. III-D);
//  4. R(i, j) = -(x^1_i + x^d_j)^T (b^1_i + b^d_j)
//            = -x^1_i^T b^1_i - x^d_j^T b^d_j - (x^1_i^T b^d_j + x^d_j^T b^1_i),
//     the m x n cross term as one product.
//
// C is symmetric but indefinite (a saddle point): H alone is indefinite,
// positive definite only on the currents that satisfy the constraints.
// The factorisation works on that subspace (null-space method): per
// interface the last TSV's current is eliminated, I^a = Z u^a + g_a e_p with
// Z = [I_{p-1}; -1^T], so H_Z = Z^T H Z ((p-1)(d-1) square, symmetric
// positive definite) takes a blocked Cholesky factorisation, u = H_Z^-1 Z^T
// (f - H E g), and the voltage differences follow from the last row of each
// interface, y_a = f_(a,p-1) - (H I)_(a,p-1).  The paper decomposes C by LU
// (its Sec. IV); the answer is the same, the symmetric positive definite
// form needs no pivoting.
//
// The dense float64 work (factorisation with the forward elimination of every
// right-hand side, back substitution, the cross-term product) runs as 64 x 64
// tiles on the float64 matrix cores (v_mfma_f64_16x16x4).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "reff_internal.h"
#include "tile_inverse.h"

namespace reff {
namespace {

constexpr int TB = 64;  // tile edge of the dense kernels

typedef double d4v __attribute__((ext_vector_type(4)));

// ---- H_Z u = rhs for all right-hand sides, 64-row panels.
//
// With Q_P = L^-T, L L^T = A_PP of panel P (after the panels before it),
// eliminating P subtracts (A_iP Q_P) (Q_P^T [A_jP^T, b_P]) from the trailing
// blocks A_ij and from the right-hand sides b_i, and u_P = Q_P Q_P^T (b_P -
// sum_{R after P} A_RP^T u_R): A_RP stays in place.  Products with the triangle
// on both sides keep Cholesky's accuracy; with A_PP^-1 between them instead (a
// product less) TSVs from 1e-6 to 1e6 ohm on one stack came out 3e-5 off,
// against 3e-11 here.  A panel is one launch each way.  A workgroup recomputes
// its two 64 x 64 operands (three times the products of kept ones, against a
// launch per panel and a pass over them), and the one that updates the next
// diagonal tile inverts its factor on the spot: the serial chain is one tile
// sweep and three tile products per panel.  4 x 512 x 512 with 512 TSVs (1533
// unknowns, 2176 right-hand sides): 1.8 ms, 7.2 ms as 164 launches of
// Cholesky, panel and update steps before.

// Loads the 64 x 64 tile at (i0, j0) of a row-major matrix (rows < M, columns
// < N; zero outside) into LDS, transposed with TR.
template <bool TR>
__device__ __forceinline__ void stage_tile(const double* __restrict__ A, int64_t lda, int i0,
                                           int j0, int M, int N, double (*T)[TB + 1]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double v[16];
  const bool cok = j0 + lane < N;
  const double* a = A + (int64_t)i0 * lda + j0 + (cok ? lane : 0);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = wv + 4 * e;
    v[e] = cok && i0 + r < M ? a[(int64_t)r * lda] : 0.0;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = wv + 4 * e;
    if (TR)
      T[lane][r] = v[e];
    else
      T[r][lane] = v[e];
  }
}

// acc = L R of two tiles in LDS (64 x 64 x 64); wave w: rows 16 w .. 16 w + 15.
__device__ __forceinline__ void tile_product(const double (*L)[TB + 1], const double (*R)[TB + 1],
                                             d4v* acc) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cc = lane & 15, kr = lane >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int ks = 0; ks < TB / 4; ++ks) {
    const double a = L[16 * w + cc][4 * ks + kr];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, R[4 * ks + kr][16 * q + cc], acc[q], 0, 0, 0);
  }
}

// Inverse of the Cholesky factor of the diagonal tile held in T (identity
// beyond its rows), transposed (upper triangular), by way of X, into Q.  The
// tile is scaled to a unit diagonal for the sweep; a pivot that is not
// positive sets *bad.
struct RootScratch {
  SweepBlock sb;
  double sc[TB];
  int drop[TB];
};
__device__ __forceinline__ void finish_diagonal(double (*T)[TB + 1], double (*X)[TB + 1],
                                                RootScratch& rs, double* __restrict__ Q, int* bad) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t < TB) rs.sc[t] = rsqrt64(T[t][t]);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) T[16 * w + r][lane] *= rs.sc[16 * w + r] * rs.sc[lane];
  __syncthreads();
  sweep_blocks<true>(T, rs.sb, 0.0, rs.drop, rs.sc, X);
  if (t < TB && rs.drop[t]) atomicOr(bad, 1);
  for (int e = t; e < TB * TB; e += 256) Q[e] = X[e >> 6][e & 63];
}

// Q[0] of panel 0.
__global__ __launch_bounds__(256) void k_chol_first(int n, const double* __restrict__ A,
                                                    double* __restrict__ Q, int* bad) {
  __shared__ double T[TB][TB + 1], X[TB][TB + 1];
  __shared__ RootScratch rs;
  const int nb = min(TB, n);
  for (int e = threadIdx.x; e < TB * TB; e += 256) {
    const int i = e >> 6, j = e & 63;
    T[i][j] = i < nb && j < nb ? A[(int64_t)i * n + j] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  finish_diagonal(T, X, rs, Q, bad);
}

__device__ __forceinline__ void store_tile(const d4v* acc, double (*T)[TB + 1]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cc = lane & 15, kr = lane >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) T[16 * w + kr + 4 * r][16 * q + cc] = acc[q][r];
}

// Eliminates panel kt (a full one: there are rows after it).  blockIdx.y =
// row tile after the panel; blockIdx.x = column tile after the panel (lower
// tiles only) or, past those, tile of the right-hand sides.
__global__ __launch_bounds__(256, 2) void k_chol_step(int n, int kt, int ntile, double* __restrict__ A,
                                                      double* __restrict__ Q, int ne,
                                                      double* __restrict__ rhs, int* bad) {
  __shared__ double S0[TB][TB + 1], S1[TB][TB + 1];
  __shared__ RootScratch rs;
  const int rest = ntile - 1 - kt, ti = kt + 1 + blockIdx.y;
  const bool mat = (int)blockIdx.x < rest;
  if (mat && blockIdx.x > blockIdx.y) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cc = lane & 15, kr = lane >> 4;
  const int p0 = kt * TB, i0 = ti * TB;
  const int j0 = mat ? (kt + 1 + (int)blockIdx.x) * TB : ((int)blockIdx.x - rest) * TB;
  const int N = mat ? n : ne;
  double* C = mat ? A : rhs;
  const double* Qp = Q + (size_t)kt * TB * TB;
  d4v wi[4], acc[4];
  stage_tile<false>(A, n, i0, p0, n, n, S0);  // A_iP Q
  stage_tile<false>(Qp, TB, 0, 0, TB, TB, S1);
  __syncthreads();
  tile_product(S0, S1, wi);
  __syncthreads();
  stage_tile<true>(Qp, TB, 0, 0, TB, TB, S0);  // Q^T X, X = A_jP^T or b_P
  if (mat)
    stage_tile<true>(A, n, j0, p0, n, n, S1);
  else
    stage_tile<false>(rhs, ne, p0, j0, n, ne, S1);
  __syncthreads();
  tile_product(S0, S1, acc);
  __syncthreads();
  store_tile(wi, S0);
  store_tile(acc, S1);
  __syncthreads();
  tile_product(S0, S1, acc);
  const bool next = mat && blockIdx.x == 0 && blockIdx.y == 0;
  if (next) __syncthreads();  // S0 becomes the next diagonal tile
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * w + kr + 4 * r, j = 16 * q + cc;
      const bool ok = i0 + i < n && j0 + j < N;
      double v = i == j ? 1.0 : 0.0;
      if (ok) {
        double* c = &C[(int64_t)(i0 + i) * N + j0 + j];
        v = *c - acc[q][r];
        *c = v;
      }
      if (next) S0[i][j] = v;
    }
  if (next) {
    __syncthreads();
    finish_diagonal(S0, S1, rs, Q + (size_t)(kt + 1) * TB * TB, bad);
  }
}

// Back substitution of panel kt: u_P = Q_P Q_P^T b_P (blockIdx.y == kt, into
// U), b_i -= A_Pi^T u_P for the row tiles i before it; blockIdx.x = tile of
// the right-hand sides.
__global__ __launch_bounds__(256, 2) void k_chol_back(int n, int kt, const double* __restrict__ A,
                                                      const double* __restrict__ Q, int ne,
                                                      double* __restrict__ rhs,
                                                      double* __restrict__ U) {
  __shared__ double S0[TB][TB + 1], S1[TB][TB + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cc = lane & 15, kr = lane >> 4;
  const int p0 = kt * TB, i0 = (int)blockIdx.y * TB, j0 = (int)blockIdx.x * TB;
  const bool own = (int)blockIdx.y == kt;
  const double* Qp = Q + (size_t)kt * TB * TB;
  stage_tile<true>(Qp, TB, 0, 0, TB, TB, S0);
  stage_tile<false>(rhs, ne, p0, j0, n, ne, S1);
  __syncthreads();
  d4v acc[4];
  tile_product(S0, S1, acc);
  __syncthreads();
  stage_tile<false>(Qp, TB, 0, 0, TB, TB, S0);
  store_tile(acc, S1);
  __syncthreads();
  tile_product(S0, S1, acc);
  if (!own) {
    __syncthreads();
    store_tile(acc, S1);
    stage_tile<true>(A, n, p0, i0, n, n, S0);  // A_Pi^T
    __syncthreads();
    tile_product(S0, S1, acc);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * w + kr + 4 * r, j = j0 + 16 * q + cc;
      if (i >= n || j >= ne) continue;
      if (own)
        U[(int64_t)i * ne + j] = acc[q][r];
      else
        rhs[(int64_t)i * ne + j] -= acc[q][r];
    }
}

// H entry between TSV k of interface b and TSV j of interface a (0-based
// interfaces a, b in [0, d-1), interface a joining tiers a and a+1):
// RT[t][j][k] = TSV-TSV resistance on tier t, rt[k][a] = segment resistance.
__device__ __forceinline__ double h_entry(const double* __restrict__ RT,
                                          const double* __restrict__ rt, int d, int p, int a,
                                          int j, int b, int k) {
  const size_t pp = (size_t)p * p;
  if (a == b) {
    double v = -0.5 * (RT[a * pp + (size_t)j * p + k] + RT[(a + 1) * pp + (size_t)j * p + k]);
    if (j == k) v += rt[(size_t)k * (d - 1) + a];
    return v;
  }
  if (b == a + 1 || a == b + 1) return 0.5 * RT[max(a, b) * pp + (size_t)j * p + k];
  return 0.0;
}

// H_Z = Z^T H Z: entry ((a, j), (b, k)), j, k < p-1, is
// H(aj, bk) - H(aj, b p-1) - H(a p-1, bk) + H(a p-1, b p-1).
__global__ __launch_bounds__(256) void k_assemble_hz(int d, int p, const double* __restrict__ RT,
                                                     const double* __restrict__ rt,
                                                     double* __restrict__ HZ) {
  const int q = p - 1, nz = q * (d - 1);
  const int64_t total = (int64_t)nz * nz;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(e / nz), c = (int)(e % nz);
    const int a = r / q, j = r % q, b = c / q, k = c % q;
    HZ[e] = h_entry(RT, rt, d, p, a, j, b, k) - h_entry(RT, rt, d, p, a, j, b, p - 1) -
            h_entry(RT, rt, d, p, a, p - 1, b, k) + h_entry(RT, rt, d, p, a, p - 1, b, p - 1);
  }
}

// Endpoint e (bumps first, then loads): f_e is -R_{s_e,.}/2 in interface
// 0 (bump) or d-2 (load), g_e = 1/2 per interface.  Reduced right-hand side
// rhs[(a,j)][e] = v(a,j) - v(a,p-1), v = f_e - H E g_e with
// (H E g)(a,j) = sum_b H(aj, b p-1) / 2.
__device__ __forceinline__ double f_entry(const double* __restrict__ Rs1,
                                          const double* __restrict__ Rsd, int d, int p, int m,
                                          int e, int a, int j) {
  if (e < m) return a == 0 ? -0.5 * Rs1[(size_t)e * p + j] : 0.0;
  return a == d - 2 ? -0.5 * Rsd[(size_t)(e - m) * p + j] : 0.0;
}

__global__ __launch_bounds__(256) void k_reduced_rhs(int d, int p, int m, int ne,
                                                     const double* __restrict__ RT,
                                                     const double* __restrict__ rt,
                                                     const double* __restrict__ Rs1,
                                                     const double* __restrict__ Rsd,
                                                     double* __restrict__ rhs) {
  const int q = p - 1, nz = q * (d - 1);
  const int64_t total = (int64_t)nz * ne;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(x / ne), e = (int)(x % ne);
    const int a = row / q, j = row % q;
    double hj = 0.0, hl = 0.0;
    for (int b = max(a - 1, 0); b <= min(a + 1, d - 2); ++b) {
      hj += h_entry(RT, rt, d, p, a, j, b, p - 1);
      hl += h_entry(RT, rt, d, p, a, p - 1, b, p - 1);
    }
    const double vj = f_entry(Rs1, Rsd, d, p, m, e, a, j) - 0.5 * hj;
    const double vl = f_entry(Rs1, Rsd, d, p, m, e, a, p - 1) - 0.5 * hl;
    rhs[x] = vj - vl;
  }
}

// From u (nz x ne): the TSV currents I_e (interface-major, p per
// interface; the last one is 1/2 - sum of the others), the voltage
// differences y_a = f(a,p-1) - (H I)(a,p-1), and per endpoint
//   selfv[e] = -x_e^T b_e - (sum_a y_e,a) / 2
// (the part of R(i,j) that depends on one endpoint only), plus the two
// operands of the cross term: crossA[i] = [I_i in interface d-2, f_i in
// interface 0] for bumps, crossB[j] = [f_j in interface d-2, I_j in
// interface 0] for loads, so that crossA_i . crossB_j = x_i^T b_j minus its
// y part + x_j^T b_i minus its y part.  One workgroup per endpoint.
__global__ __launch_bounds__(256) void k_reduced_post(int d, int p, int m, int ne,
                                                      const double* __restrict__ RT,
                                                      const double* __restrict__ rt,
                                                      const double* __restrict__ Rs1,
                                                      const double* __restrict__ Rsd,
                                                      const double* __restrict__ U,
                                                      double* __restrict__ Icur,
                                                      double* __restrict__ selfv,
                                                      double* __restrict__ crossA,
                                                      double* __restrict__ crossB) {
  const int e = blockIdx.x, t = threadIdx.x;
  const int q = p - 1, K = p * (d - 1);
  double* I = Icur + (size_t)e * K;
  __shared__ double red[256];
  __shared__ double ysum_s, self_s;
  // currents
  for (int a = 0; a < d - 1; ++a) {
    double s = 0.0;
    for (int j = t; j < q; j += 256) {
      const double u = U[(size_t)(a * q + j) * ne + e];
      I[a * p + j] = u;
      s += u;
    }
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (t < h) red[t] += red[t + h];
      __syncthreads();
    }
    if (t == 0) I[a * p + q] = 0.5 - red[0];
    __syncthreads();
  }
  __threadfence_block();
  __syncthreads();
  if (t == 0) ysum_s = 0.0, self_s = 0.0;
  __syncthreads();
  // y_a and the two dot products of x_e^T b_e
  for (int a = 0; a < d - 1; ++a) {
    double s = 0.0;
    for (int b = max(a - 1, 0); b <= min(a + 1, d - 2); ++b)
      for (int k = t; k < p; k += 256) s += h_entry(RT, rt, d, p, a, q, b, k) * I[b * p + k];
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (t < h) red[t] += red[t + h];
      __syncthreads();
    }
    if (t == 0) {
      const double y = f_entry(Rs1, Rsd, d, p, m, e, a, q) - red[0];
      ysum_s += y;
    }
    __syncthreads();
  }
  {
    double s = 0.0;
    for (int a = 0; a < d - 1; ++a)
      for (int k = t; k < p; k += 256) s += I[a * p + k] * f_entry(Rs1, Rsd, d, p, m, e, a, k);
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (t < h) red[t] += red[t + h];
      __syncthreads();
    }
  }
  if (t == 0) {
    // x_e^T b_e = I^T f + y^T g, g = 1/2 per interface
    const double xb = red[0] + 0.5 * ysum_s;
    selfv[e] = -xb - 0.5 * ysum_s;
  }
  for (int k = t; k < p; k += 256) {
    if (e < m) {
      double* A = crossA + (size_t)e * 2 * p;
      A[k] = I[(d - 2) * p + k];
      A[p + k] = f_entry(Rs1, Rsd, d, p, m, e, 0, k);
    } else {
      double* B = crossB + (size_t)(e - m) * 2 * p;
      B[k] = f_entry(Rs1, Rsd, d, p, m, e, d - 2, k);
      B[p + k] = I[k];
    }
  }
}

// Cross term: G[z] = A B^T over part z of the 64-column steps of K (A m x K,
// B n x K), one 64 x 64 tile per workgroup.  A step is one tile product, its
// 32 loads per thread in flight together, and K is split until the launch has
// CROSS_WORKGROUPS: 128 x 2048 pairs over K = 1024 are 64 tiles only, 200 us
// with 16 columns at a time and one part, now 18 us.
constexpr int CROSS_WORKGROUPS = 512;

int cross_parts(int64_t m, int64_t n, int p) {
  const int64_t tiles = ((m + TB - 1) / TB) * ((n + TB - 1) / TB);
  const int64_t steps = (2 * (int64_t)p + TB - 1) / TB;
  return (int)std::max<int64_t>(1, std::min(steps, CROSS_WORKGROUPS / tiles));
}

__global__ __launch_bounds__(256, 2) void k_cross(int m, int n, int K, const double* __restrict__ A,
                                                  const double* __restrict__ B,
                                                  double* __restrict__ G) {
  __shared__ double S0[TB][TB + 1], S1[TB][TB + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, cc = lane & 15, kr = lane >> 4;
  const int i0 = blockIdx.y * TB, j0 = blockIdx.x * TB;
  const int steps = (K + TB - 1) / TB, z = blockIdx.z, parts = gridDim.z;
  d4v acc[4], sum[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) sum[q] = d4v{0.0, 0.0, 0.0, 0.0};
  for (int k = steps * z / parts; k < steps * (z + 1) / parts; ++k) {
    __syncthreads();
    stage_tile<false>(A, K, i0, k * TB, m, K, S0);
    stage_tile<true>(B, K, j0, k * TB, n, K, S1);
    __syncthreads();
    tile_product(S0, S1, acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[q] += acc[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * w + kr + 4 * r, j = j0 + 16 * q + cc;
      if (i < m && j < n) G[((int64_t)z * m + i) * n + j] = sum[q][r];
    }
}

// R(i, j) = selfv[i] + selfv[m + j] - sum of the parts of G[i][j].
__global__ __launch_bounds__(256) void k_reduced_finish(int m, int n, int parts,
                                                        const double* __restrict__ selfv,
                                                        const double* __restrict__ G,
                                                        double* __restrict__ out) {
  const int64_t total = (int64_t)m * n;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(x / n), j = (int)(x % n);
    double g = G[x];
    for (int z = 1; z < parts; ++z) g += G[z * total + x];
    out[x] = selfv[i] + selfv[m + j] - g;
  }
}

dim3 rgrid(int64_t n) { return dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)); }

// Device memory of one call: the arrays are named first, then carved from
// one allocation.
struct Carve {
  struct Part {
    void** p;
    size_t bytes;
  };
  std::vector<Part> parts;
  char* base = nullptr;
  template <typename T>
  void add(T** out, size_t count) {
    parts.push_back(Part{(void**)out, (std::max<size_t>(count, 1) * sizeof(T) + 255) / 256 * 256});
  }
  hipError_t alloc() {
    size_t total = 0;
    for (const Part& q : parts) total += q.bytes;
    const hipError_t e = hipMalloc((void**)&base, total);
    if (e != hipSuccess) return e;
    char* at = base;
    for (const Part& q : parts) {
      *q.p = at;
      at += q.bytes;
    }
    return hipSuccess;
  }
  ~Carve() {
    if (base) (void)hipFree(base);
  }
};

}  // namespace
}  // namespace reff

extern "C" reff_status reff_reduced_pairs(int32_t n_tiers, int32_t nx, int32_t ny,
                                          const double* r_t, const double* s_t, int32_t p,
                                          const int32_t* tsv_xy, const double* tsv_r, int64_t m,
                                          const int32_t* bump_xy, int64_t n,
                                          const int32_t* load_xy, double* R_out,
                                          int32_t out_on_device, void* stream) try {
  using namespace reff;
  const int d = n_tiers;
  if (d < 2) return host_fail(REFF_ERR_INVALID_ARG, "the reduced system needs at least 2 tiers");
  if (nx < 1 || ny < 1) return host_fail(REFF_ERR_INVALID_ARG, "tier size must be at least 1 x 1");
  if (p < 1) return host_fail(REFF_ERR_INVALID_ARG, "at least one TSV column is needed");
  if (m < 0 || n < 0) return host_fail(REFF_ERR_INVALID_ARG, "negative bump or load count");
  if (!r_t || !s_t || !tsv_xy || !tsv_r)
    return host_fail(REFF_ERR_INVALID_ARG, "NULL tier or TSV array");
  if (m * n == 0) return REFF_OK;
  if (!bump_xy || !load_xy || !R_out) return host_fail(REFF_ERR_INVALID_ARG, "NULL bump, load or output");
  for (int t = 0; t < d; ++t)
    if (!std::isfinite(r_t[t]) || !(r_t[t] > 0.0) || !std::isfinite(s_t[t]) || !(s_t[t] > 0.0))
      return host_fail(REFF_ERR_INVALID_ARG, "tier edge resistances must be finite and positive");
  for (int64_t k = 0; k < (int64_t)p * (d - 1); ++k)
    if (!std::isfinite(tsv_r[k]) || !(tsv_r[k] > 0.0))
      return host_fail(REFF_ERR_INVALID_ARG, "TSV segment resistances must be finite and positive");
  auto on_grid = [&](const int32_t* xy, int64_t cnt) {
    for (int64_t k = 0; k < cnt; ++k)
      if (xy[2 * k] < 0 || xy[2 * k] >= nx || xy[2 * k + 1] < 0 || xy[2 * k + 1] >= ny) return false;
    return true;
  };
  if (!on_grid(tsv_xy, p) || !on_grid(bump_xy, m) || !on_grid(load_xy, n))
    return host_fail(REFF_ERR_INVALID_ARG, "a TSV, bump or load is off the tier grid");
  {
    std::vector<int64_t> ids(p);
    for (int k = 0; k < p; ++k) ids[k] = (int64_t)tsv_xy[2 * k + 1] * nx + tsv_xy[2 * k];
    std::sort(ids.begin(), ids.end());
    if (std::adjacent_find(ids.begin(), ids.end()) != ids.end())
      return host_fail(REFF_ERR_INVALID_ARG, "duplicate TSV column");
  }
  const int64_t P0 = p + m, Pd = p + n;
  if (P0 > 65535 || Pd > 65535)
    return host_fail(REFF_ERR_INVALID_ARG, "at most 65535 TSVs plus bumps (or loads) per call");
  hipStream_t st = (hipStream_t)stream;
  auto dev_fail = [&](hipError_t e, const char* what) {
    return host_fail(e == hipErrorOutOfMemory ? REFF_ERR_OUT_OF_MEMORY : REFF_ERR_DEVICE,
                     std::string(what) + ": " + hipGetErrorString(e));
  };
  const int q = p - 1, nz = q * (d - 1), ne = (int)(m + n);
  const int ntile = (nz + TB - 1) / TB;
  const int parts = cross_parts(m, n, p);
  // the cosine tables of all tiers, or (few endpoints on a very large tier, or
  // no room for the tables) direct products tier by tier through a P x P array
  const size_t Pm = (size_t)std::max(P0, Pd);
  int32_t* dxy = nullptr;
  double* drs = nullptr;
  char* tab = nullptr;
  double *dR = nullptr, *RT = nullptr, *rt = nullptr, *Rs1 = nullptr, *Rsd = nullptr;
  double *HZ = nullptr, *Q = nullptr, *rhs = nullptr, *U = nullptr;
  double *Icur = nullptr, *selfv = nullptr, *cA = nullptr, *cB = nullptr, *G = nullptr;
  double* dout = nullptr;
  int* bad = nullptr;
  Carve mem;
  auto arrays = [&](bool with_table) {
    mem.parts.clear();
    mem.add(&dxy, 2 * (size_t)(p + m + n));
    mem.add(&drs, 2 * (size_t)d);
    if (with_table)
      mem.add(&tab, grid_tiers_bytes(nx, ny, d));
    else
      mem.add(&dR, Pm * Pm);
    mem.add(&RT, (size_t)d * p * p);
    mem.add(&rt, (size_t)p * (d - 1));
    mem.add(&Rs1, (size_t)m * p);
    mem.add(&Rsd, (size_t)n * p);
    mem.add(&HZ, (size_t)nz * nz);
    mem.add(&Q, (size_t)ntile * TB * TB);
    mem.add(&rhs, (size_t)nz * ne);
    mem.add(&U, (size_t)nz * ne);
    mem.add(&Icur, (size_t)ne * p * (d - 1));
    mem.add(&selfv, (size_t)ne);
    mem.add(&cA, (size_t)m * 2 * p);
    mem.add(&cB, (size_t)n * 2 * p);
    mem.add(&G, (size_t)parts * m * n);
    mem.add(&bad, 1);
    if (!out_on_device) mem.add(&dout, (size_t)m * n);
  };
  bool table = grid_use_table(nx, ny, (int64_t)Pm);
  arrays(table);
  hipError_t e = mem.alloc();
  if (e == hipErrorOutOfMemory && table) {
    (void)hipGetLastError();
    table = false;
    arrays(false);
    e = mem.alloc();
  }
  if (e != hipSuccess) return dev_fail(e, "hipMalloc");
  double* out = out_on_device ? R_out : dout;
  // (a fill kernel of the runtime; the call is never captured, it synchronises)
  e = hipMemsetAsync(bad, 0, sizeof(int), st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(rt, tsv_r, sizeof(double) * p * (d - 1), hipMemcpyHostToDevice, st);
  // 1. intra-die resistances: TSV-TSV of every tier, bump-TSV of tier 0,
  //    load-TSV of the last tier
  std::vector<int32_t> pts;
  std::vector<double> rs;
  if (table && e == hipSuccess) {
    pts.assign(tsv_xy, tsv_xy + 2 * (size_t)p);
    pts.insert(pts.end(), bump_xy, bump_xy + 2 * m);
    pts.insert(pts.end(), load_xy, load_xy + 2 * n);
    std::vector<GridRect> rects;
    for (int t = 0; t < d; ++t) {
      rs.push_back(r_t[t]);
      rs.push_back(s_t[t]);
      rects.push_back(GridRect{t, dxy, dxy, p, p, RT + (size_t)t * p * p});
    }
    rects.push_back(GridRect{0, dxy + 2 * (size_t)p, dxy, m, p, Rs1});
    rects.push_back(GridRect{d - 1, dxy + 2 * (size_t)(p + m), dxy, n, p, Rsd});
    e = hipMemcpyAsync(dxy, pts.data(), sizeof(int32_t) * pts.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
      e = hipMemcpyAsync(drs, rs.data(), sizeof(double) * rs.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
      e = grid_tiers_launch(nx, ny, d, drs, rects.data(), (int)rects.size(), tab, st);
  }
  for (int t = 0; !table && t < d && e == hipSuccess; ++t) {
    pts.assign(tsv_xy, tsv_xy + 2 * (size_t)p);
    int64_t extra = 0;
    if (t == 0) pts.insert(pts.end(), bump_xy, bump_xy + 2 * m), extra = m;
    if (t == d - 1) pts.insert(pts.end(), load_xy, load_xy + 2 * n), extra = n;
    const int64_t P = p + extra;
    e = hipMemcpyAsync(dxy, pts.data(), sizeof(int32_t) * 2 * P, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = grid_pairs_device(nx, ny, r_t[t], s_t[t], dxy, P, dR, st);
    if (e == hipSuccess)
      e = hipMemcpy2DAsync(RT + (size_t)t * p * p, sizeof(double) * p, dR, sizeof(double) * P,
                           sizeof(double) * p, p, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && extra > 0)
      e = hipMemcpy2DAsync(t == 0 ? Rs1 : Rsd, sizeof(double) * p, dR + (size_t)p * P,
                           sizeof(double) * P, sizeof(double) * p, extra,
                           hipMemcpyDeviceToDevice, st);
    // the staged points are read by the next tier's upload only after
    // this tier's kernels have run
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  // 2.-3. H_Z, its Cholesky factor, and the reduced solves for all endpoints
  if (e == hipSuccess && nz > 0) {
    hipLaunchKernelGGL(k_assemble_hz, rgrid((int64_t)nz * nz), dim3(256), 0, st, d, p,
                       (const double*)RT, (const double*)rt, HZ);
    e = hipGetLastError();
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_reduced_rhs, rgrid((int64_t)nz * ne), dim3(256), 0, st, d, p,
                         (int)m, ne, (const double*)RT, (const double*)rt, (const double*)Rs1,
                         (const double*)Rsd, rhs);
      e = hipGetLastError();
    }
    if (e == hipSuccess) {
      hipLaunchKernelGGL(k_chol_first, dim3(1), dim3(256), 0, st, nz, (const double*)HZ, Q, bad);
      e = hipGetLastError();
    }
    const unsigned et = (unsigned)((ne + TB - 1) / TB);
    for (int kt = 0; kt + 1 < ntile && e == hipSuccess; ++kt) {
      const unsigned rest = (unsigned)(ntile - 1 - kt);
      hipLaunchKernelGGL(k_chol_step, dim3(rest + et, rest), dim3(256), 0, st, nz, kt, ntile, HZ, Q,
                         ne, rhs, bad);
      e = hipGetLastError();
    }
    for (int kt = ntile - 1; kt >= 0 && e == hipSuccess; --kt) {
      hipLaunchKernelGGL(k_chol_back, dim3(et, (unsigned)(kt + 1)), dim3(256), 0, st, nz, kt,
                         (const double*)HZ, (const double*)Q, ne, rhs, U);
      e = hipGetLastError();
    }
  }
  // 4. currents, voltage differences, self terms, cross-term operands
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_reduced_post, dim3((unsigned)ne), dim3(256), 0, st, d, p, (int)m, ne,
                       (const double*)RT, (const double*)rt, (const double*)Rs1,
                       (const double*)Rsd, (const double*)U, Icur, selfv, cA, cB);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_cross, dim3((unsigned)((n + TB - 1) / TB), (unsigned)((m + TB - 1) / TB),
                                     (unsigned)parts),
                       dim3(256), 0, st, (int)m, (int)n, 2 * p, (const double*)cA,
                       (const double*)cB, G);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_reduced_finish, rgrid(m * n), dim3(256), 0, st, (int)m, (int)n, parts,
                       (const double*)selfv, (const double*)G, out);
    e = hipGetLastError();
  }
  if (e == hipSuccess && !out_on_device)
    e = hipMemcpyAsync(R_out, dout, sizeof(double) * m * n, hipMemcpyDeviceToHost, st);
  int hbad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return dev_fail(e, "reduced pairs");
  if (hbad)
    return host_fail(REFF_ERR_DEVICE,
                     "reduced system: a pivot of Z^T H Z was not positive");
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}
