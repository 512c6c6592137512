// Internal declarations of the screening model (surrogate_api.cpp and
// surrogate_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/reff_surrogate.h"

namespace reffsg {

// Screening support for reff_batch_plans: whether a plan has the model's
// geometry, and the predicted R of every node of n plans into the device
// buffer R [n][n_tiers*ny*nx] (pads 0), on stream st.
bool geometry_matches(reff_surrogate s, const reff_pdn_desc* d);
reff_status predict_device(reff_surrogate s, const reff_pdn_desc* plans, int32_t n, double* R,
                           hipStream_t st);

// A 3x3 (taps 9, zero padding) or 1x1 (taps 1) convolution over P = B H W
// pixels as a product on the matrix cores (BF16 inputs, FP32 accumulation):
//   C(p, n) = relu?(sum over k = tap cin + c < K of X[p + tap][c] Wn[n][k] + bias[n])
// stored as FP32 or BF16 at C[p ldc + n]; with up = c > 0 (a 2x2 transposed
// convolution of c channels, N = 4 c) column (a 2 + b) c + ch of pixel (y, x)
// is stored at channel ch of pixel (2 y + a, 2 x + b).  Rows of Wn hold
// conv_row(K) values, zero past K.
struct ConvArgs {
  const uint16_t* X;
  int64_t ldx;
  int cin, taps, P, H, W;
  const uint16_t* Wn;
  int N, K;
  const float* bias;
  int relu;
  void* C;
  int64_t ldc;
  int c_fp32, up;
  int magic;  // set by conv
};
constexpr int64_t conv_row(int64_t K) { return (K + 31) / 32 * 32; }

// Weight gradient of such a convolution: out[m][n] = sum_p X[p + tap][c]
// dY[p][n], m = tap cin + c (`part`: room for the partial sums).
struct WgradArgs {
  const uint16_t* X;
  int64_t ldx;
  int cin, taps, P, H, W;
  const uint16_t* dY;
  int64_t ldy;
  int N;
  float* part;
  int chunk, magic;  // set by wgrad
};

// One labelled node of a training batch: pixel (b*H + y)*W + x of the
// batch, tier t, target log R.
struct LabelRec {
  int32_t pix;
  int32_t t;
  float logR;
  float pad_;
};

hipError_t conv(ConvArgs g, hipStream_t st);
hipError_t wgrad(WgradArgs g, float* out, int64_t part_floats, hipStream_t st);
hipError_t pool_fwd(const uint16_t* X, int64_t ldx, int C, int B, int H, int W, uint16_t* Y,
                    hipStream_t st);
// dX (row stride ldx) += dY routed to the first maximum of each 2x2 window
hipError_t pool_bwd(const uint16_t* X, int64_t ldx, const uint16_t* dY, int C, int B, int H,
                    int W, uint16_t* dX, hipStream_t st);
// space-to-depth: S[(b, y, x)][(a*2+c)*C + ch] = Y[(b, 2y+a, 2x+c)][ch]; H, W
// are the low-resolution sizes
hipError_t s2d(const uint16_t* Y, int64_t ldy, int C, int B, int H, int W, uint16_t* S,
               hipStream_t st);
// dY *= (Y > 0) over P rows of C channels
hipError_t relu_bwd(uint16_t* dY, int64_t lddy, const uint16_t* Y, int64_t ldy, int C, int64_t P,
                    hipStream_t st);
// db[c] = sum over P rows of dY[p][c]; part holds nblk*C floats
hipError_t colsum(const uint16_t* dY, int64_t ld, int C, int64_t P, float* part, int nblk,
                  float* db, hipStream_t st);
// BF16 copies of W [(kh*K + kw)*Cin + ci][co] for the products: Wb[co][(kh*K +
// kw)*Cin + ci] and, for the input gradient, the flipped taps Wt[ci][((K-1-kh)*K
// + (K-1-kw))*Cout + co]; rows of conv_row values
hipError_t weight_copies(const float* W, int Cin, int Cout, int K, uint16_t* Wb, uint16_t* Wt,
                         hipStream_t st);
// dpred[pix][t] = 2 (pred - logR) / n for each label (dpred zeroed first);
// part[blockIdx] = partial sums of (pred - logR)^2
hipError_t masked_loss(const float* pred, int nt, const LabelRec* lab, int n, float inv_n,
                       uint16_t* dpred, double* part, int nblk, hipStream_t st);
hipError_t adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                float b2, float eps, float bc1, float bc2, hipStream_t st);
hipError_t fill16(uint16_t* a, int64_t n, uint16_t val, hipStream_t st);
// R[(b*nt + t)*H*W + y*W + x] = pad ? 0 : exp(pred[((b*H + y)*W + x)*nt + t]);
// padm is the pad mask [b][H*W] (1 = pad)
hipError_t predict_out(const float* pred, const uint8_t* padm, int B, int nt, int H, int W,
                       double* R, hipStream_t st);

}  // namespace reffsg
