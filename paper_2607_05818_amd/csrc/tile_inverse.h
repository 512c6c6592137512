// Inverse of one 64 x 64 symmetric positive definite tile by a workgroup of
// four waves (device code shared by the sparse-direct fronts and the reduced
// pair system).
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
// panel of the root of the 4 x 512 x 512 stack: 25 us, where Cholesky and the
// triangular inverse took 101 us and their repetition in the inversion 60 us.
__device__ __forceinline__ void invert_tile(double (*T)[TILE + 1], double (*Cp)[17], int w, int* bad) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int cc = lane & 15, kr = lane >> 4;
  for (int b = 0; 16 * b < w; ++b) {
    if (wv == 0) {
      double a[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) a[c] = T[lane][16 * b + c];
      bool ok = true;
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const int q = 16 * b + p;  // pivot row and column
        const double piv = lane_value(a[p], q);
        ok = ok && piv > 0.0 && std::isfinite(piv);
        const double inv = 1.0 / piv;
        // row q becomes inv * row q, row r loses (a_rp inv) * row q
        const double mult = lane == q ? inv : -a[p] * inv;
        const double keep = lane == q ? 0.0 : 1.0;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          if (c == p) continue;
          const double s = lane_value(a[c], q);
          a[c] = fma(mult, s, a[c] * keep);
        }
        a[p] = mult;
      }
      if (!ok && lane == 0) atomicOr(bad, 1);
#pragma unroll
      for (int c = 0; c < 16; ++c) Cp[lane][c] = a[c];
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
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(
            Cp[16 * wv + cc][4 * ks + kr], T[16 * b + 4 * ks + kr][16 * j + cc], acc[j], 0, 0, 0);
    }
    __syncthreads();  // every strip has read row block b
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        T[16 * wv + kr + 4 * r][16 * j + cc] =
            j == b ? Cp[16 * wv + kr + 4 * r][cc] : acc[j][r];
    __syncthreads();
  }
}

}  // namespace reff
