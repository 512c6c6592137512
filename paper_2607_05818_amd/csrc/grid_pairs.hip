// Two-point resistances on a uniform M x N resistor grid by the closed form
// of Eq. 3 (Sec. II-B), for every pair of a point set: the intra-die
// resistances of the paper's divide-and-conquer pair method (Sec. III-C/D).
//
// For points (x1, y1), (x2, y2), with xh = x + 1/2, yh = y + 1/2,
//   R = r |x1 - x2| / N + s |y1 - y2| / M
//       + 2 / (M N) sum_{m=1}^{M-1} sum_{n=1}^{N-1}
//           (cos(m t xh1) cos(n u yh1) - cos(m t xh2) cos(n u yh2))^2
//           / ((1 - cos(m t)) / r + (1 - cos(n u)) / s),
// t = pi / M, u = pi / N.  With T_ij the sum of cos(m t xh_i) cos(m t xh_j)
// cos(n u yh_i) cos(n u yh_j) W[m][n] (W the reciprocal denominator), the
// double sum of a pair is T_ii + T_jj - 2 T_ij.
//
// Cosine table (k_grid_tables, k_grid_cos_gemm, k_grid_rect).  A product of
// cosines is half the sum of the cosines of the difference and of the sum of
// the angles, and the points are integers, so
//   T_ij = (F(dx, dy) + F(dx, sy) + F(sx, dy) + F(sx, sy)) / 4,
//   F(a, b) = sum_mn W[m][n] cos(pi m a / M) cos(pi n b / N),
// dx = |x_i - x_j|, sx = x_i + x_j + 1 (folded at M, dy and sy alike): one
// (M+1) x (N+1) table, two matrix products over W, serves every pair of the
// tier.
//
// Direct products (k_grid_gram), for few points on a very large tier: T = X
// diag(W) X^T over K = (M-1)(N-1) on the float64 matrix cores, its m factors
// from the multiple-angle recurrence cos((m+1) a) = 2 cos(a) cos(m a) -
// cos((m-1) a) as in the paper's GPU evaluation (Sec. III-D); k_grid_finish
// forms R.
#include <hip/hip_runtime.h>
#include <cmath>
#include <stdint.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "reff_internal.h"

namespace reff {
namespace {

// W[(m-1)(N-1) + n-1] = 1 / ((1 - cos(m t)) / r + (1 - cos(n u)) / s).
__global__ __launch_bounds__(256) void k_grid_weights(int M, int N, double r, double s,
                                                      double* __restrict__ W) {
  const int64_t total = (int64_t)(M - 1) * (N - 1);
  const double t = M_PI / M, u = M_PI / N;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int m = (int)(q / (N - 1)) + 1, n = (int)(q % (N - 1)) + 1;
    W[q] = 1.0 / ((1.0 - cos(m * t)) / r + (1.0 - cos(n * u)) / s);
  }
}

// k_grid_gram computes 64 x 64 blocks of T (upper block pairs only) on the
// float64 matrix cores (16x16x4), the K range split over workgroups by m
// segment; its operands are formed on the fly: the n factor from a table C[p][n-1] =
// cos(n u yh_p) staged in LDS per 64-wide chunk of n, the m factor from the
// multiple-angle recurrence per lane, W from the weight table.  Each
// segment writes its partial block; k_grid_finish sums them and forms R.
constexpr int GG_B = 64;    // points per block
constexpr int GG_NC = 64;   // n values per staged chunk
// Time of a product of the direct path over one of the table's, near the line
// between them (see grid_use_table).
constexpr double DIRECT_COST = 0.5;

__global__ __launch_bounds__(256) void k_grid_ncos(int N, const int32_t* __restrict__ xy,
                                                   int64_t P, double* __restrict__ Cn) {
  const int64_t total = P * (N - 1);
  const double u = M_PI / N;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = q / (N - 1);
    const int n = (int)(q % (N - 1)) + 1;
    Cn[q] = cos(n * u * (xy[2 * p + 1] + 0.5));
  }
}

// Grid (block pairs, m segments).  Tpart[seg][i][j] for the block pair's
// i, j (rows of block bi, columns of block bj, bi <= bj); points past P
// are stand-ins (the last point) whose entries are not written.
__global__ __launch_bounds__(256) void k_grid_gram(int M, int N, const int32_t* __restrict__ xy,
                                                   const double* __restrict__ W,
                                                   const double* __restrict__ Cn, int64_t P,
                                                   int nb, int mseg, double* __restrict__ Tpart) {
  __shared__ double BI[GG_B][GG_NC + 1], BJ[GG_B][GG_NC + 1];
  int q = blockIdx.x, bi = 0;
  while (q >= nb - bi) q -= nb - bi, ++bi;
  const int bj = bi + q;
  const int seg = blockIdx.y;
  const int mlen = (M - 1 + mseg - 1) / mseg;
  const int m0 = 1 + seg * mlen, m1 = min(M, m0 + mlen);  // m in [m0, m1)
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int cc = lane & 15, kr = lane >> 4;
  const double t = M_PI / M;
  const int64_t ia = min((int64_t)bi * GG_B + w * 16 + cc, P - 1);
  int64_t jb[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) jb[tt] = min((int64_t)bj * GG_B + tt * 16 + cc, P - 1);
  const double xi = xy[2 * ia] + 0.5;
  double xj[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) xj[tt] = xy[2 * jb[tt]] + 0.5;
  typedef double d4 __attribute__((ext_vector_type(4)));
  d4 acc[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) acc[tt] = d4{0.0, 0.0, 0.0, 0.0};
  for (int n0 = 1; n0 < N; n0 += GG_NC) {
    __syncthreads();  // the previous chunk is no longer read
    for (int e = threadIdx.x; e < GG_B * GG_NC; e += blockDim.x) {
      const int pt = e / GG_NC, k = e % GG_NC, n = n0 + k;
      const int64_t pi = min((int64_t)bi * GG_B + pt, P - 1), pj = min((int64_t)bj * GG_B + pt, P - 1);
      const bool ok = n < N;
      BI[pt][k] = ok ? Cn[pi * (N - 1) + (n - 1)] : 0.0;
      BJ[pt][k] = ok ? Cn[pj * (N - 1) + (n - 1)] : 0.0;
    }
    __syncthreads();
    if (m0 >= m1) continue;
    // cos(m a) at m = m0 and m0 - 1, then the recurrence
    double ai = cos(m0 * t * xi), pi_ = cos((m0 - 1) * t * xi), ki = 2.0 * cos(t * xi);
    double aj[4], pj_[4], kj[4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      aj[tt] = cos(m0 * t * xj[tt]);
      pj_[tt] = cos((m0 - 1) * t * xj[tt]);
      kj[tt] = 2.0 * cos(t * xj[tt]);
    }
    for (int m = m0; m < m1; ++m) {
      const double* Wm = W + (int64_t)(m - 1) * (N - 1);
#pragma unroll 4  // (full unrolling needs 305 registers: one wave per SIMD)
      for (int ks = 0; ks < GG_NC / 4; ++ks) {
        const int k = 4 * ks + kr, n = n0 + k;
        const double wv = Wm[min(n, N - 1) - 1];
        const double A = ai * BI[w * 16 + cc][k];
        const double wk = n < N ? wv : 0.0;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          const double B = wk * aj[tt] * BJ[tt * 16 + cc][k];
          acc[tt] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, B, acc[tt], 0, 0, 0);
        }
      }
      const double qi = fma(ki, ai, -pi_);
      pi_ = ai, ai = qi;
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        const double qj = fma(kj[tt], aj[tt], -pj_[tt]);
        pj_[tt] = aj[tt], aj[tt] = qj;
      }
    }
  }
  double* Ts = Tpart + (int64_t)seg * P * P;
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i = (int64_t)bi * GG_B + w * 16 + kr + 4 * r;
      const int64_t j = (int64_t)bj * GG_B + tt * 16 + cc;
      if (i < P && j < P) Ts[i * P + j] = acc[tt][r];
    }
}

// R(i,j) from the summed partial T (its upper blocks): r |dx| / N + s |dy| / M
// + 2 / (M N) (T_ii + T_jj - 2 T_ij), i != j; R(i,i) = 0.  T_ij is read at
// (min, max), so both halves of R are the same value.
__global__ __launch_bounds__(256) void k_grid_finish(int M, int N, double r, double s,
                                                     const int32_t* __restrict__ xy,
                                                     const double* __restrict__ Tpart,
                                                     int mseg, int64_t P,
                                                     double* __restrict__ out) {
  const int64_t total = P * P;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = q / P, j = q % P;
    if (i == j) {
      out[q] = 0.0;
      continue;
    }
    const int64_t lo = min(i, j), hi = max(i, j);
    double tii = 0.0, tjj = 0.0, tij = 0.0;
    for (int g = 0; g < mseg; ++g) {
      const double* Ts = Tpart + (int64_t)g * P * P;
      tii += Ts[lo * P + lo];
      tjj += Ts[hi * P + hi];
      tij += Ts[lo * P + hi];
    }
    const int dx = xy[2 * lo] - xy[2 * hi], dy = xy[2 * lo + 1] - xy[2 * hi + 1];
    out[q] = r * fabs((double)dx) / N + s * fabs((double)dy) / M +
             2.0 / ((double)M * N) * (tii + tjj - 2.0 * tij);
  }
}

// Cosine table of nt tiers that share their size (edge resistances rs[2 t]
// along x and rs[2 t + 1] along y).  Per tier: A holds the first product,
// (M+1) x (N-1), and F the table, (M+1) x (N+1); F's memory holds W, (M-1) x
// (N-1), until the second product overwrites it.
struct GridTables {
  double* cx;  // cos(pi q / M), q < 2 M (shared by the tiers)
  double* cy;  // cos(pi q / N), q < 2 N
  double* A;
  double* F;
};

// cx, cy and every tier's W (as k_grid_weights).
__global__ __launch_bounds__(256) void k_grid_tables(int M, int N, int nt,
                                                     const double* __restrict__ rs, GridTables g) {
  const int64_t nw = (int64_t)(M - 1) * (N - 1), nf = (int64_t)(M + 1) * (N + 1);
  const int64_t ncos = 2 * (int64_t)M + 2 * (int64_t)N, total = ncos + nt * nw;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * blockDim.x) {
    if (q < 2 * (int64_t)M) {
      g.cx[q] = cospi((double)q / M);
    } else if (q < ncos) {
      g.cy[q - 2 * (int64_t)M] = cospi((double)(q - 2 * (int64_t)M) / N);
    } else {
      const int t = (int)((q - ncos) / nw);
      const int64_t e = (q - ncos) % nw;
      const int m = (int)(e / (N - 1)) + 1, n = (int)(e % (N - 1)) + 1;
      g.F[t * nf + e] =
          1.0 / ((1.0 - cos(m * (M_PI / M))) / rs[2 * t] + (1.0 - cos(n * (M_PI / N))) / rs[2 * t + 1]);
    }
  }
}

// One of the table's two products, blockIdx.z = tier:
//   SECOND = false:  A[a][n] = sum_m cos(pi m a / M) W[m][n],  a <= M
//   SECOND = true:   F[a][b] = sum_n A[a][n] cos(pi n b / N),  a <= M, b <= N
// on v_mfma_f64_16x16x4, one 32 x 32 output tile per workgroup, a 16 x 16
// quarter per wave (a 512 x 512 tier has 289 tiles: with 64 x 64 tiles most
// of the 256 CUs would stand idle); K goes through LDS 32 at a time, the next
// slice's loads in flight while the matrix cores work.  The cosine operand
// is cos(pi (k l mod 2 L) / L) from the table of 2 L values: a thread keeps
// the residues of its elements and steps them by 32 l mod 2 L per slice, so
// no angle is ever larger than 2 pi and no product of indices overflows.
// LDS rows are padded to 34 doubles (the 16 lanes of a quarter-wave read 16
// rows at one k).  Every pair of 256 points of a 512 x 512 tier, the whole
// call: 635 us by direct products, 72 us by the table (work memory in place).
template <bool SECOND>
__global__ __launch_bounds__(256) void k_grid_cos_gemm(int M, int N, GridTables g) {
  constexpr int T = 32;
  __shared__ double sA[T][T + 2], sB[T][T + 2];  // [row][k], [column][k]
  const int64_t nf = (int64_t)(M + 1) * (N + 1), na = (int64_t)(M + 1) * (N - 1);
  const int K = (SECOND ? N : M) - 1, cols = SECOND ? N + 1 : N - 1;
  const int L2 = 2 * (SECOND ? N : M);  // period of the cosine operand
  const double* tab = SECOND ? g.cy : g.cx;
  const double* dense = SECOND ? g.A + blockIdx.z * na : g.F + blockIdx.z * nf;
  const int i0 = blockIdx.y * T, j0 = blockIdx.x * T;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int cc = lane & 15, kr = lane >> 4, wi = 16 * (w >> 1), wj = 16 * (w & 1);
  // this thread's four elements of each operand slice: the cosine operand at
  // index l (row a or column b) and k = t & 31, the dense one along its rows
  int res[4], step[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int l = min((SECOND ? j0 : i0) + (t >> 5) + 8 * e, SECOND ? N : M);
    res[e] = (int)((int64_t)((t & 31) + 1) * l % L2);
    step[e] = (int)((int64_t)T * l % L2);
  }
  double rc[4], rd[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      rc[e] = k0 + (t & 31) < K ? tab[res[e]] : 0.0;
      res[e] += step[e];
      if (res[e] >= L2) res[e] -= L2;
      if (SECOND) {  // A[row][k], k along the lanes
        const int a = i0 + (t >> 5) + 8 * e, k = k0 + (t & 31);
        rd[e] = a <= M && k < K ? dense[(int64_t)a * (N - 1) + k] : 0.0;
      } else {  // W[k][column], columns along the lanes
        const int k = k0 + (t >> 5) + 8 * e, n = j0 + (t & 31);
        rd[e] = k < K && n < cols ? dense[(int64_t)k * (N - 1) + n] : 0.0;
      }
    }
  };
  typedef double d4 __attribute__((ext_vector_type(4)));
  d4 acc = d4{0.0, 0.0, 0.0, 0.0};
  if (K > 0) load(0);
  for (int k0 = 0; k0 < K; k0 += T) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = (t >> 5) + 8 * e, k = t & 31;
      if (SECOND) {
        sB[r][k] = rc[e];
        sA[r][k] = rd[e];
      } else {
        sA[r][k] = rc[e];
        sB[k][r] = rd[e];
      }
    }
    __syncthreads();
    if (k0 + T < K) load(k0 + T);
#pragma unroll
    for (int ks = 0; ks < T / 4; ++ks)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sA[wi + cc][4 * ks + kr], sB[wj + cc][4 * ks + kr],
                                                 acc, 0, 0, 0);
  }
  double* out = SECOND ? g.F + blockIdx.z * nf : g.A + blockIdx.z * na;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int a = i0 + wi + kr + 4 * r, j = j0 + wj + cc;
    if (a <= M && j < cols) out[(int64_t)a * cols + j] = acc[r];
  }
}

// 4 T_ij from the table.
__device__ __forceinline__ double grid_t4(const double* __restrict__ F, int M, int N, int xi,
                                          int yi, int xj, int yj) {
  const int dx = abs(xi - xj), dy = abs(yi - yj);
  const int sx = min(xi + xj + 1, 2 * M - (xi + xj + 1)), sy = min(yi + yj + 1, 2 * N - (yi + yj + 1));
  const double* f0 = F + (int64_t)dx * (N + 1);
  const double* f1 = F + (int64_t)sx * (N + 1);
  return (f0[dy] + f1[dy]) + (f0[sy] + f1[sy]);
}

// R(i, j) of the row points xyr[0 .. nr) and the column points xyc[0 .. nc)
// of one tier: r |dx| / N + s |dy| / M + (2 / (M N)) (T_ii + T_jj - 2 T_ij).
// Every term is symmetric in the two points, and 4 T_ij is 4 T_ii where they
// coincide, so R is exactly symmetric and exactly 0 there.  blockIdx.y walks
// the rows, a workgroup's lanes the columns; the table (2 MB at 512 x 512)
// stays in L2.
__global__ __launch_bounds__(256) void k_grid_rect(int M, int N, const double* __restrict__ rs,
                                                   const int32_t* __restrict__ xyr, int64_t nr,
                                                   const int32_t* __restrict__ xyc, int64_t nc,
                                                   const double* __restrict__ F,
                                                   double* __restrict__ out) {
  const double cx = rs[0] / N, cy = rs[1] / M, c4 = 0.5 / ((double)M * N);
  for (int64_t i = blockIdx.y; i < nr; i += gridDim.y) {
    const int xi = xyr[2 * i], yi = xyr[2 * i + 1];
    const double ti = grid_t4(F, M, N, xi, yi, xi, yi);
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nc;
         j += (int64_t)gridDim.x * blockDim.x) {
      const int xj = xyc[2 * j], yj = xyc[2 * j + 1];
      const double tj = grid_t4(F, M, N, xj, yj, xj, yj);
      const double tij = grid_t4(F, M, N, xi, yi, xj, yj);
      out[i * nc + j] =
          cx * abs(xi - xj) + cy * abs(yi - yj) + c4 * ((ti + tj) - 2.0 * tij);
    }
  }
}

// The four launches of the direct products: weights, cosines, Gram blocks, R.
hipError_t grid_direct_launch(int M, int N, double r, double s, const int32_t* dxy, int64_t P,
                             double* dW, double* dC, double* dT, int mseg, double* o,
                             hipStream_t st) {
  const int64_t nb = (P + GG_B - 1) / GG_B;
  const int64_t nbp = nb * (nb + 1) / 2;
  const size_t nw = (size_t)(M - 1) * (N - 1);
  const size_t ncos = (size_t)P * (N - 1);
  auto grid1 = [](size_t n) { return dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)); };
  hipError_t e = hipSuccess;
  if (nw > 0) {
    hipLaunchKernelGGL(k_grid_weights, grid1(nw), dim3(256), 0, st, M, N, r, s, dW);
    e = hipGetLastError();
  }
  if (e == hipSuccess && ncos > 0) {
    hipLaunchKernelGGL(k_grid_ncos, grid1(ncos), dim3(256), 0, st, N, dxy, P, dC);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_grid_gram, dim3((unsigned)nbp, (unsigned)mseg), dim3(256), 0, st, M, N,
                       dxy, (const double*)dW, (const double*)dC, P, (int)nb, mseg, dT);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_grid_finish, grid1((size_t)P * P), dim3(256), 0, st, M, N, r, s, dxy,
                       (const double*)dT, mseg, P, o);
    e = hipGetLastError();
  }
  return e;
}

// Segments of the m range: about 2048 workgroups per launch.
int grid_pairs_mseg(int M, int64_t P) {
  const int64_t nb = (P + GG_B - 1) / GG_B;
  const int64_t nbp = nb * (nb + 1) / 2;
  return (int)std::max<int64_t>(1, std::min<int64_t>(std::max(M - 1, 1), (2048 + nbp - 1) / nbp));
}

size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

// The table's launches for nt tiers of one size: cosines and W, the two
// products.  k_grid_rect then reads F.
hipError_t grid_table_launch(int M, int N, int nt, const double* drs, const GridTables& g,
                             hipStream_t st) {
  auto tiles = [](int64_t n) { return (unsigned)((n + 31) / 32); };
  const int64_t total = 2 * (int64_t)M + 2 * (int64_t)N + nt * (int64_t)(M - 1) * (N - 1);
  hipLaunchKernelGGL(k_grid_tables, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 4096)),
                     dim3(256), 0, st, M, N, nt, drs, g);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_grid_cos_gemm<false>, dim3(tiles(N - 1), tiles(M + 1), nt), dim3(256), 0,
                       st, M, N, g);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_grid_cos_gemm<true>, dim3(tiles(N + 1), tiles(M + 1), nt), dim3(256), 0,
                       st, M, N, g);
    e = hipGetLastError();
  }
  return e;
}

hipError_t grid_rect_launch(int M, int N, const double* drs, const int32_t* xyr, int64_t nr,
                            const int32_t* xyc, int64_t nc, const double* F, double* out,
                            hipStream_t st) {
  if (nr <= 0 || nc <= 0) return hipSuccess;
  const dim3 grid((unsigned)std::min<int64_t>((nc + 255) / 256, 1024),
                  (unsigned)std::min<int64_t>(nr, 65535));
  hipLaunchKernelGGL(k_grid_rect, grid, dim3(256), 0, st, M, N, drs, xyr, nr, xyc, nc, F, out);
  return hipGetLastError();
}

// Bytes of the table's arrays for nt tiers, in the order they are carved:
// cosines, A, F.
size_t grid_table_bytes(int M, int N, int nt) {
  return round256(sizeof(double) * 2 * (size_t)M) + round256(sizeof(double) * 2 * (size_t)N) +
         round256(sizeof(double) * nt * (size_t)(M + 1) * std::max(N - 1, 0)) +
         round256(sizeof(double) * nt * (size_t)(M + 1) * (N + 1));
}

GridTables grid_table_carve(char* base, int M, int N, int nt) {
  GridTables g;
  g.cx = (double*)base;
  base += round256(sizeof(double) * 2 * (size_t)M);
  g.cy = (double*)base;
  base += round256(sizeof(double) * 2 * (size_t)N);
  g.A = (double*)base;
  base += round256(sizeof(double) * nt * (size_t)(M + 1) * std::max(N - 1, 0));
  g.F = (double*)base;
  return g;
}

reff_status grid_pairs_validate(int32_t M, int32_t N, double r, double s, const int32_t* xy,
                                int64_t P, const double* R_out) {
  if (M < 1 || N < 1) return host_fail(REFF_ERR_INVALID_ARG, "grid size must be at least 1 x 1");
  if (!std::isfinite(r) || !(r > 0.0) || !std::isfinite(s) || !(s > 0.0))
    return host_fail(REFF_ERR_INVALID_ARG, "edge resistances must be finite and positive");
  if (P < 0) return host_fail(REFF_ERR_INVALID_ARG, "negative point count");
  if (P == 0) return REFF_OK;
  if (!xy || !R_out) return host_fail(REFF_ERR_INVALID_ARG, "NULL points or output");
  if (P > 65535) return host_fail(REFF_ERR_INVALID_ARG, "at most 65535 points per call");
  for (int64_t k = 0; k < P; ++k)
    if (xy[2 * k] < 0 || xy[2 * k] >= M || xy[2 * k + 1] < 0 || xy[2 * k + 1] >= N)
      return host_fail(REFF_ERR_INVALID_ARG, "point " + std::to_string(k) + " is off the grid");
  return REFF_OK;
}

reff_status grid_dev_fail(hipError_t e, const char* what) {
  return host_fail(e == hipErrorOutOfMemory ? REFF_ERR_OUT_OF_MEMORY : REFF_ERR_DEVICE,
                   std::string(what) + ": " + hipGetErrorString(e));
}

// Work memory of reff_grid_pairs_noalloc: one array per GPU, resident until
// the process ends.  Host code never passes `scratch` itself to a kernel or
// a copy (on the host it is only a stand-in for the symbol); it uses the
// device address looked up once per device below.
constexpr size_t kScratchBytes = (size_t)64 << 20;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace
}  // namespace reff

namespace reff {

// Which path serves P points of an M x N tier.  Both are float64
// matrix-core products; the table does (M+1)(N-1)(M+N) of them whatever P
// is, the direct products (M-1)(N-1) for each entry of the padded upper
// block pairs.  At 512 x 512 a product costs the direct path twice the
// table's time, at 2048 x 2048 the same, at 4096 x 4096 (whose operands no
// longer stay in L2 for the table's 32 x 32 tiles) half.  The two are near
// each other only on tiers of that size, so a direct product counts half:
// table / direct measured 0.10 / 0.64 ms at 512 x 512 and 256 points, 0.12 /
// 0.27 ms at 16 points, 1.5 / 1.5 ms at 2048 x 2048 and 64 points, 13.2 / 9.9
// ms at 4096 x 4096 and 65 points.
// On one-wide tiers every sum is empty and the direct kernels do no work; the
// table's launch grid and doubled coordinates bound M and N.
bool grid_use_table(int M, int N, int64_t P) {
  if (M < 2 || N < 2 || M > (1 << 20) || N > (1 << 20)) return false;
  auto pad = [](int64_t n, int64_t t) { return (double)((n + t - 1) / t * t); };
  const int64_t nb = (P + GG_B - 1) / GG_B;
  const double table = pad(M + 1, 32) * (pad(N - 1, 32) * (M - 1) + pad(N + 1, 32) * (N - 1));
  const double direct = 0.5 * nb * (nb + 1) * GG_B * GG_B * (M - 1) * pad(N - 1, GG_NC);
  return table <= DIRECT_COST * direct;
}

// Tiers that share one launch: as many as 8 GiB of tables hold, and as a grid
// has in z (65535).
static int grid_tier_group(int M, int N, int nt) {
  const size_t nf = (size_t)(M + 1) * (N + 1);
  const size_t most = std::min<size_t>(65535, ((size_t)8 << 30) / (16 * nf));
  return (int)std::min<size_t>(nt, std::max<size_t>(1, most));
}

size_t grid_tiers_bytes(int M, int N, int nt) {
  return grid_table_bytes(M, N, grid_tier_group(M, N, nt));
}

hipError_t grid_tiers_launch(int M, int N, int nt, const double* drs, const GridRect* rects,
                             int nrect, char* work, hipStream_t st) {
  const size_t nf = (size_t)(M + 1) * (N + 1);
  const int ng = grid_tier_group(M, N, nt);
  hipError_t e = hipSuccess;
  for (int t0 = 0; t0 < nt && e == hipSuccess; t0 += ng) {
    const int cnt = std::min(ng, nt - t0);
    const GridTables g = grid_table_carve(work, M, N, cnt);
    e = grid_table_launch(M, N, cnt, drs + 2 * t0, g, st);
    for (int k = 0; k < nrect && e == hipSuccess; ++k) {
      const GridRect& q = rects[k];
      if (q.tier < t0 || q.tier >= t0 + cnt) continue;
      e = grid_rect_launch(M, N, drs + 2 * q.tier, q.xyr, q.nr, q.xyc, q.nc,
                           g.F + (q.tier - t0) * nf, q.out, st);
    }
  }
  return e;
}

// All-pairs Eq. 3 resistances of P points already in device memory, by the
// direct products, into device out[P * P]; the work memory is allocated here
// and released after the stream has run the kernels (the call returns with
// them complete).
hipError_t grid_pairs_device(int M, int N, double r, double s, const int32_t* dxy, int64_t P,
                             double* dout, hipStream_t st) {
  if (P <= 0) return hipSuccess;
  const int mseg = grid_pairs_mseg(M, P);
  double *dW = nullptr, *dC = nullptr, *dT = nullptr;
  hipError_t e = hipMalloc((void**)&dW, std::max<size_t>((size_t)(M - 1) * (N - 1), 1) * sizeof(double));
  if (e == hipSuccess)
    e = hipMalloc((void**)&dC, std::max<size_t>((size_t)P * (N - 1), 1) * sizeof(double));
  if (e == hipSuccess) e = hipMalloc((void**)&dT, (size_t)mseg * P * P * sizeof(double));
  if (e == hipSuccess) e = grid_direct_launch(M, N, r, s, dxy, P, dW, dC, dT, mseg, dout, st);
  const hipError_t e2 = hipStreamSynchronize(st);
  if (e == hipSuccess) e = e2;
  if (dW) (void)hipFree(dW);
  if (dC) (void)hipFree(dC);
  if (dT) (void)hipFree(dT);
  return e;
}

namespace {

// Points and edge resistances of a one-tier call, as uploaded: r, s, then
// the points (in one copy).
std::vector<char> grid_inputs(double r, double s, const int32_t* xy, int64_t P) {
  std::vector<char> h(2 * sizeof(double) + (size_t)P * 2 * sizeof(int32_t));
  const double rs[2] = {r, s};
  std::memcpy(h.data(), rs, sizeof(rs));
  std::memcpy(h.data() + sizeof(rs), xy, (size_t)P * 2 * sizeof(int32_t));
  return h;
}

// One call on work memory laid out as inputs, then (host output) the
// staging of R, then the table's arrays.
size_t grid_call_bytes(int M, int N, int64_t P, bool out_on_device) {
  return round256(2 * sizeof(double) + (size_t)P * 2 * sizeof(int32_t)) +
         (out_on_device ? 0 : round256((size_t)P * P * sizeof(double))) + grid_table_bytes(M, N, 1);
}

hipError_t grid_table_call(int M, int N, double r, double s, const int32_t* xy, int64_t P,
                           double* R_out, bool out_on_device, char* base, hipStream_t st) {
  const std::vector<char> h = grid_inputs(r, s, xy, P);
  const double* drs = (const double*)base;
  const int32_t* dxy = (const int32_t*)(base + 2 * sizeof(double));
  hipError_t e = hipMemcpyAsync(base, h.data(), h.size(), hipMemcpyHostToDevice, st);
  base += round256(h.size());
  double* o = R_out;
  if (!out_on_device) {
    o = (double*)base;
    base += round256((size_t)P * P * sizeof(double));
  }
  const GridTables g = grid_table_carve(base, M, N, 1);
  if (e == hipSuccess) e = grid_table_launch(M, N, 1, drs, g, st);
  if (e == hipSuccess) e = grid_rect_launch(M, N, drs, dxy, P, dxy, P, g.F, o, st);
  if (e == hipSuccess && !out_on_device)
    e = hipMemcpyAsync(R_out, o, (size_t)P * P * sizeof(double), hipMemcpyDeviceToHost, st);
  // also where a launch failed: the staged inputs and the work memory go
  const hipError_t e2 = hipStreamSynchronize(st);
  return e == hipSuccess ? e2 : e;
}

}  // namespace
}  // namespace reff

extern "C" reff_status reff_grid_pairs(int32_t M, int32_t N, double r, double s,
                                       const int32_t* xy, int64_t P, double* R_out,
                                       int32_t out_on_device, void* stream) try {
  using namespace reff;
  const reff_status v = grid_pairs_validate(M, N, r, s, xy, P, R_out);
  if (v != REFF_OK || P == 0) return v;
  hipStream_t st = (hipStream_t)stream;
  if (grid_use_table(M, N, P)) {
    char* base = nullptr;
    hipError_t e = hipMalloc((void**)&base, grid_call_bytes(M, N, P, out_on_device));
    if (e == hipSuccess) {
      e = grid_table_call(M, N, r, s, xy, P, R_out, out_on_device, base, st);
      (void)hipFree(base);
      return e == hipSuccess ? REFF_OK : grid_dev_fail(e, "grid pairs");
    }
    if (e != hipErrorOutOfMemory) return grid_dev_fail(e, "hipMalloc");
    (void)hipGetLastError();  // no room for the table: the direct products
  }
  const int mseg = grid_pairs_mseg(M, P);
  const size_t nw = (size_t)(M - 1) * (N - 1);
  const size_t ncos = (size_t)P * (N - 1);
  const size_t tbytes = (size_t)mseg * P * P * sizeof(double);
  const size_t obytes = (size_t)P * P * sizeof(double);
  int32_t* dxy = nullptr;
  double *dW = nullptr, *dC = nullptr, *dT = nullptr, *dout = nullptr;
  auto release = [&]() {
    if (dxy) (void)hipFree(dxy);
    if (dW) (void)hipFree(dW);
    if (dC) (void)hipFree(dC);
    if (dT) (void)hipFree(dT);
    if (dout) (void)hipFree(dout);
  };
  hipError_t e = hipMalloc((void**)&dxy, (size_t)P * 2 * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc((void**)&dW, std::max<size_t>(nw, 1) * sizeof(double));
  if (e == hipSuccess) e = hipMalloc((void**)&dC, std::max<size_t>(ncos, 1) * sizeof(double));
  if (e == hipSuccess) e = hipMalloc((void**)&dT, tbytes);
  if (e == hipSuccess && !out_on_device) e = hipMalloc((void**)&dout, obytes);
  if (e != hipSuccess) {
    release();
    return grid_dev_fail(e, "hipMalloc");
  }
  double* o = out_on_device ? R_out : dout;
  e = hipMemcpyAsync(dxy, xy, (size_t)P * 2 * sizeof(int32_t), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = grid_direct_launch(M, N, r, s, dxy, P, dW, dC, dT, mseg, o, st);
  if (e == hipSuccess && !out_on_device)
    e = hipMemcpyAsync(R_out, dout, obytes, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  release();
  if (e != hipSuccess) return grid_dev_fail(e, "grid pairs");
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}

extern "C" reff_status reff_grid_pairs_noalloc(int32_t M, int32_t N, double r, double s,
                                               const int32_t* xy, int64_t P, double* R_out,
                                               int32_t out_on_device, void* stream) try {
  using namespace reff;
  const reff_status v = grid_pairs_validate(M, N, r, s, xy, P, R_out);
  if (v != REFF_OK || P == 0) return v;
  // Layout of the work memory: points, weights, cosine table, host staging
  // of R (host output only), then as many m segments of partial Gram blocks
  // as fit, up to the count the allocating entry point uses.
  const size_t b_xy = round256((size_t)P * 2 * sizeof(int32_t));
  const size_t b_w = round256((size_t)(M - 1) * (N - 1) * sizeof(double));
  const size_t b_c = round256((size_t)P * (N - 1) * sizeof(double));
  const size_t b_o = out_on_device ? 0 : round256((size_t)P * P * sizeof(double));
  const size_t b_seg = (size_t)P * P * sizeof(double);
  const size_t fixed = b_xy + b_w + b_c + b_o;
  if (fixed + b_seg > kScratchBytes)
    return host_fail(REFF_ERR_INVALID_ARG,
                     "grid pairs without allocation: " + std::to_string(M) + " x " +
                         std::to_string(N) + " with " + std::to_string(P) + " points needs " +
                         std::to_string(fixed + b_seg) + " bytes of work memory, more than the " +
                         std::to_string(kScratchBytes) + " bytes it holds");
  const int mseg = (int)std::min<size_t>(grid_pairs_mseg(M, P), (kScratchBytes - fixed) / b_seg);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return grid_dev_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return host_fail(REFF_ERR_UNSUPPORTED, "device index too large");
  unsigned char* base = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void* ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return grid_dev_fail(e, "hipGetSymbolAddress(scratch)");
      g_scratch_ptr[dev] = ptr;
    }
    base = (unsigned char*)g_scratch_ptr[dev];
  }
  hipStream_t st = (hipStream_t)stream;
  // The table's arrays need about two tiers of doubles where the direct
  // products need one and the points' cosines: calls that only the latter
  // fit keep taking them.
  if (grid_use_table(M, N, P) && grid_call_bytes(M, N, P, out_on_device) <= kScratchBytes) {
    e = grid_table_call(M, N, r, s, xy, P, R_out, out_on_device, (char*)base, st);
    return e == hipSuccess ? REFF_OK : grid_dev_fail(e, "grid pairs (no allocation)");
  }
  int32_t* dxy = (int32_t*)base;
  double* dW = (double*)(base + b_xy);
  double* dC = (double*)(base + b_xy + b_w);
  double* dout = (double*)(base + b_xy + b_w + b_c);
  double* dT = (double*)(base + fixed);
  double* o = out_on_device ? R_out : dout;
  e = hipMemcpyAsync(dxy, xy, (size_t)P * 2 * sizeof(int32_t), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = grid_direct_launch(M, N, r, s, dxy, P, dW, dC, dT, mseg, o, st);
  if (e == hipSuccess && !out_on_device)
    e = hipMemcpyAsync(R_out, dout, (size_t)P * P * sizeof(double), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return grid_dev_fail(e, "grid pairs (no allocation)");
  return REFF_OK;
} catch (...) {
  return reff::host_exception();
}
