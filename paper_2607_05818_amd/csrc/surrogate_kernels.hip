// gfx950 kernels of the screening model: BF16 matrix-core products that carry
// every convolution (implicit GEMMs: the 3x3 neighbourhoods are read where
// they lie; the 2x2 transposed convolution is a 1x1 product whose rows are
// stored depth-to-space), plus the pooling, layout, loss and optimiser kernels
// around them.  Activations are NHWC BF16 (stored as uint16_t), accumulation
// is FP32.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "surrogate_internal.h"

namespace reffsg {

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));

constexpr int BK = 32;       // K step of the convolution product
constexpr int LDT = BK + 8;  // LDS row pitch: 16 rows of 16 bytes on 64 banks

// K index -> tap without a division (magic = 2^20 / cin + 1): k / cin while k
// cin < 2^20, which holds for every layer whose channels are no multiple of 8
// (at most 254) and for the first 32 k of the others.
__device__ __forceinline__ int tap_of(int k, int magic) { return (int)(((int64_t)k * magic) >> 20); }

// C(p, n) = sum over taps and channels of X[p shifted by the tap][c] W[n][k],
// k = tap cin + c: the convolution as a product over K = taps x cin whose A
// rows are formed by the loads (taps outside the image are zero).  A workgroup
// of four waves makes 64 MR pixels x NT channels, a wave 16 MR x NT of them
// as MR x NT / 16 tiles of v_mfma_f32_16x16x32_bf16, K ascending in steps of
// 32 (the instruction adds its k in order: the sums are those of the 16-wide
// form bit for bit).  A thread moves eight consecutive k (one tap, for cin a
// multiple of 8) of MR rows and of one row of W per step with 16-byte loads;
// the next step's are in flight while the current products run, and the LDS
// tiles are double-buffered, so one barrier per step suffices.
// Bound by LDS reads (MR + NT / 16 per MR NT / 16 products); MR = 4 where that
// leaves at least two workgroups per CU, else MR = 1.
// At 16 plans of 3 x 128 x 128 (C = 32) the kernels of a forward pass take 575
// us; with im2col copies, 64 x 64 tiles of the 16-wide instruction and a
// depth-to-space pass they took 1,250 us.
template <int MR, int NT>
__global__ __launch_bounds__(256) void k_conv(ConvArgs g) {
  constexpr int ROWS = 64 * MR, NQ = NT / 16;
  __shared__ __align__(16) uint16_t sA[2][ROWS][LDT];
  __shared__ __align__(16) uint16_t sB[2][NT][LDT];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int p0 = blockIdx.x * ROWS, n0 = blockIdx.y * NT;
  const int row = t >> 2, kg = 8 * (t & 3);  // this thread's rows are row + 64 i
  const bool vec = g.cin % 8 == 0 && g.ldx % 8 == 0 && ((uintptr_t)g.X & 15) == 0;
  int px[MR], py[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) {
    const int p = p0 + row + 64 * i;
    px[i] = p % g.W;
    py[i] = p < g.P ? (p / g.W) % g.H : -4;  // rows past the end: no tap is inside
  }
  const int kp = (g.K + BK - 1) / BK * BK;  // rows of W are zero from K to kp
  int tap = tap_of(kg, g.magic), ci = kg - tap * g.cin;
  u4v va[MR], vb;
  auto load_step = [&](int k0) {
    if (vec) {
      const int dy = g.taps == 9 ? ((tap * 11) >> 5) - 1 : 0;
      const int dx = g.taps == 9 ? tap - 3 * (dy + 1) - 1 : 0;
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        const int y = py[i] + dy, x = px[i] + dx;
        const int64_t p = p0 + row + 64 * i + dy * g.W + dx;
        va[i] = tap < g.taps && y >= 0 && y < g.H && x >= 0 && x < g.W
                    ? *reinterpret_cast<const u4v*>(g.X + p * g.ldx + ci)
                    : u4v{0u, 0u, 0u, 0u};
      }
      ci += BK;
      while (ci >= g.cin) ci -= g.cin, ++tap;
    } else {
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        uint16_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = k0 + kg + e, tp = tap_of(k, g.magic), c = k - tp * g.cin;
          const int dy = g.taps == 9 ? ((tp * 11) >> 5) - 1 : 0;
          const int dx = g.taps == 9 ? tp - 3 * (dy + 1) - 1 : 0;
          const int y = py[i] + dy, x = px[i] + dx;
          const int64_t p = p0 + row + 64 * i + dy * g.W + dx;
          h[e] = k < g.K && y >= 0 && y < g.H && x >= 0 && x < g.W ? g.X[p * g.ldx + c] : (uint16_t)0;
        }
        va[i] = u4v{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                    (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
      }
    }
    if (row < NT)
      vb = n0 + row < g.N ? *reinterpret_cast<const u4v*>(g.Wn + (int64_t)(n0 + row) * kp + k0 + kg)
                          : u4v{0u, 0u, 0u, 0u};
  };
  auto store_step = [&](int buf) {
#pragma unroll
    for (int i = 0; i < MR; ++i) *reinterpret_cast<u4v*>(&sA[buf][row + 64 * i][kg]) = va[i];
    if (row < NT) *reinterpret_cast<u4v*>(&sB[buf][row][kg]) = vb;
  };
  f4v acc[MR][NQ];
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int j = 0; j < NQ; ++j) acc[i][j] = f4v{0.f, 0.f, 0.f, 0.f};
  load_step(0);
  store_step(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < kp; k0 += BK) {
    const bool more = k0 + BK < kp;
    if (more) load_step(k0 + BK);
    const int kc = 8 * (lane >> 4), r = lane & 15;
    b8v bf[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) bf[j] = *reinterpret_cast<const b8v*>(&sB[buf][16 * j + r][kc]);
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      const b8v af = *reinterpret_cast<const b8v*>(&sA[buf][16 * (MR * w + i) + r][kc]);
#pragma unroll
      for (int j = 0; j < NQ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf[j], acc[i][j], 0, 0, 0);
    }
    if (more) store_step(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int p = p0 + 16 * (MR * w + i) + 4 * (lane >> 4) + r;
      if (p >= g.P) continue;
      const int x = g.up ? p % g.W : 0, yb = g.up ? p / g.W : 0;  // yb = b H + y
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const int n = n0 + 16 * j + (lane & 15);
        if (n >= g.N) continue;
        float v = acc[i][j][r];
        if (g.bias) v += g.bias[n];
        if (g.relu) v = fmaxf(v, 0.f);
        int64_t at = (int64_t)p * g.ldc + n;
        if (g.up) {  // channel (a 2 + c) up + ch of pixel (y, x) goes to (2 y + a, 2 x + c)
          const int q = n / g.up;
          at = ((int64_t)(2 * yb + (q >> 1)) * (2 * g.W) + 2 * x + (q & 1)) * g.ldc + n - q * g.up;
        }
        if (g.c_fp32)
          ((float*)g.C)[at] = v;
        else
          ((uint16_t*)g.C)[at] = f2bf(v);
      }
    }
}

hipError_t conv(ConvArgs g, hipStream_t st) {
  if (g.P <= 0 || g.N <= 0) return hipSuccess;
  g.magic = (1 << 20) / g.cin + 1;
  const int nt = g.N <= 32 ? 32 : 64;
  auto blocks = [&](int rows, int n) { return dim3((g.P + rows - 1) / rows, (g.N + n - 1) / n); };
  const dim3 big = blocks(256, nt);
  if ((int64_t)big.x * big.y >= 512) {
    if (nt == 32)
      hipLaunchKernelGGL((k_conv<4, 32>), big, dim3(256), 0, st, g);
    else
      hipLaunchKernelGGL((k_conv<4, 64>), big, dim3(256), 0, st, g);
    return hipGetLastError();
  }
  const dim3 sm = blocks(64, 64);
  if (nt == 64 && (int64_t)sm.x * sm.y >= 512)
    hipLaunchKernelGGL((k_conv<1, 64>), sm, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL((k_conv<1, 32>), blocks(64, 32), dim3(256), 0, st, g);
  return hipGetLastError();
}

// Weight gradient: part[z][m][n] = sum over the pixels p of slice z of
// X[p shifted by the tap of m][channel of m] dY[p][n], m = tap cin + c.  The
// K index of the product is the pixel, along which neither operand is
// contiguous: a thread loads eight channels (16 bytes) of four consecutive
// pixels and stores them transposed, 8 bytes (four pixels) per channel, into
// the [channel][pixel] tiles that the matrix cores read.  64 x 64 tiles of
// (m, n), 64 pixels per step, wave w the quarter (w / 2, w % 2).
// Replaces an im2col copy and 2-byte LDS stores: at 16 plans of 3 x 128 x 128
// all kernels of a training step take 2.7 ms (this one 0.82), 7.4 ms before.
constexpr int GP = 64;       // pixels per step
constexpr int LGP = GP + 8;  // LDS pitch

__global__ __launch_bounds__(256) void k_wgrad(WgradArgs g) {
  __shared__ __align__(16) uint16_t sX[2][64][LGP], sD[2][64][LGP];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
  const int pbeg = blockIdx.z * g.chunk, pend = min(g.P, pbeg + g.chunk);
  const bool isx = t < 128;
  const int pg = 4 * (t & 15), cg = 8 * ((t & 127) >> 4);  // pixel and channel group
  // operand of this thread: X at (tap, c) of m, or dY at column n
  const int m = m0 + cg, n = n0 + cg;
  const int K = g.taps * g.cin;
  const int64_t ld = isx ? g.ldx : g.ldy;
  const bool vec = isx ? g.cin % 8 == 0 && g.ldx % 8 == 0 && ((uintptr_t)g.X & 15) == 0
                       : g.ldy % 8 == 0 && ((uintptr_t)g.dY & 15) == 0 && n + 8 <= g.N;
  const int tap0 = isx ? min(m, K) / g.cin : 0;
  const int wy = 64 / g.W, wx = 64 % g.W;  // one step further, in rows and columns
  int x = (pbeg + pg) % g.W, y = ((pbeg + pg) / g.W) % g.H;
  u4v v[4];
  auto load_step = [&](int p0) {
    int xx = x, yy = y;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = p0 + pg + j;
      v[j] = u4v{0u, 0u, 0u, 0u};
      if (p < pend) {
        if (vec) {
          const int dy = g.taps == 9 && isx ? ((tap0 * 11) >> 5) - 1 : 0;
          const int dx = g.taps == 9 && isx ? tap0 - 3 * (dy + 1) - 1 : 0;
          const bool in = isx ? m < K && yy + dy >= 0 && yy + dy < g.H && xx + dx >= 0 && xx + dx < g.W
                              : true;
          const uint16_t* src = isx ? g.X + ((int64_t)p + dy * g.W + dx) * ld + (m - tap0 * g.cin)
                                    : g.dY + (int64_t)p * ld + n;
          if (in) v[j] = *reinterpret_cast<const u4v*>(src);
        } else {
          uint16_t h[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            h[e] = 0;
            if (isx && m + e < K) {
              const int tp = tap_of(m + e, g.magic), c = m + e - tp * g.cin;
              const int dy = g.taps == 9 ? ((tp * 11) >> 5) - 1 : 0;
              const int dx = g.taps == 9 ? tp - 3 * (dy + 1) - 1 : 0;
              if (yy + dy >= 0 && yy + dy < g.H && xx + dx >= 0 && xx + dx < g.W)
                h[e] = g.X[((int64_t)p + dy * g.W + dx) * ld + c];
            } else if (!isx && n + e < g.N) {
              h[e] = g.dY[(int64_t)p * ld + n + e];
            }
          }
          v[j] = u4v{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                     (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
        }
      }
      if (++xx == g.W) {
        xx = 0;
        if (++yy == g.H) yy = 0;
      }
    }
    x += wx;
    y += wy;
    if (x >= g.W) x -= g.W, ++y;
    while (y >= g.H) y -= g.H;
  };
  auto store_step = [&](int buf) {
    uint16_t(*T)[LGP] = isx ? sX[buf] : sD[buf];
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // channels 2 e and 2 e + 1
      const uint32_t a = v[0][e], b = v[1][e], c = v[2][e], d = v[3][e];
      *reinterpret_cast<uint64_t*>(&T[cg + 2 * e][pg]) =
          (uint64_t)((a & 0xffffu) | (b << 16)) | ((uint64_t)((c & 0xffffu) | (d << 16)) << 32);
      *reinterpret_cast<uint64_t*>(&T[cg + 2 * e + 1][pg]) =
          (uint64_t)((a >> 16) | (b & 0xffff0000u)) | ((uint64_t)((c >> 16) | (d & 0xffff0000u)) << 32);
    }
  };
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  f4v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f4v{0.f, 0.f, 0.f, 0.f};
  if (pbeg < pend) {
    load_step(pbeg);
    store_step(0);
  }
  __syncthreads();
  int buf = 0;
  for (int p0 = pbeg; p0 < pend; p0 += GP) {
    const bool more = p0 + GP < pend;
    if (more) load_step(p0 + GP);
#pragma unroll
    for (int kk = 0; kk < GP; kk += 32) {
      const int kc = kk + 8 * (lane >> 4), r = lane & 15;
      b8v af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = *reinterpret_cast<const b8v*>(&sX[buf][wm + 16 * i + r][kc]);
        bf[i] = *reinterpret_cast<const b8v*>(&sD[buf][wn + 16 * i + r][kc]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    if (more) store_step(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  float* C = g.part + (int64_t)blockIdx.z * K * g.N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mm = m0 + wm + 16 * i + 4 * (lane >> 4) + r, nn = n0 + wn + 16 * j + (lane & 15);
        if (mm < K && nn < g.N) C[(int64_t)mm * g.N + nn] = acc[i][j][r];
      }
}

// out[i] = sum over z < nsplit of part[z len + i]: 64 entries per workgroup,
// its four waves each a quarter of the slices.
__global__ __launch_bounds__(256) void k_sum_slices(const float* __restrict__ part, int nsplit,
                                                    int64_t len, float* __restrict__ out) {
  __shared__ float red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float s = 0.f;
  if (i < len)
#pragma unroll 4
    for (int z = w; z < nsplit; z += 4) s += part[z * len + i];
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && i < len) out[i] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

hipError_t sum_slices(const float* part, int nsplit, int64_t len, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_sum_slices, dim3((unsigned)((len + 63) / 64)), dim3(256), 0, st, part, nsplit,
                     len, out);
  return hipGetLastError();
}

// Pixels of a step's slice: enough workgroups to fill the chip twice, slices
// of at least 512 pixels, and partials within part_floats.
hipError_t wgrad(WgradArgs g, float* out, int64_t part_floats, hipStream_t st) {
  const int K = g.taps * g.cin;
  const int64_t len = (int64_t)K * g.N;
  const int64_t tiles = (int64_t)((K + 63) / 64) * ((g.N + 63) / 64);
  int64_t nz = std::max<int64_t>(1, std::min<int64_t>({(1024 + tiles - 1) / tiles, g.P / 512,
                                                       part_floats / len}));
  g.chunk = (int)(((g.P + nz - 1) / nz + GP - 1) / GP * GP);
  nz = (g.P + g.chunk - 1) / g.chunk;
  g.magic = (1 << 20) / g.cin + 1;
  float* part = g.part;
  if (nz == 1) g.part = out;
  hipLaunchKernelGGL(k_wgrad, dim3((K + 63) / 64, (g.N + 63) / 64, (unsigned)nz), dim3(256), 0, st, g);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && nz > 1) e = sum_slices(part, (int)nz, len, out, st);
  return e;
}

static int blocks_for(int64_t n, int per = 256, int cap = 16384) {
  const int64_t b = (n + per - 1) / per;
  return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

__global__ void k_pool_fwd(const uint16_t* X, int64_t ldx, int C, int B, int H, int W,
                           uint16_t* Y) {
  const int Ho = H / 2, Wo = W / 2;
  const int64_t total = (int64_t)B * Ho * Wo * C;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const int64_t p = e / C;
    const int x = (int)(p % Wo);
    const int y = (int)((p / Wo) % Ho);
    const int64_t b = p / ((int64_t)Wo * Ho);
    const int64_t base = (b * H + 2 * y) * W + 2 * x;
    float m = bf2f(X[base * ldx + c]);
    m = fmaxf(m, bf2f(X[(base + 1) * ldx + c]));
    m = fmaxf(m, bf2f(X[(base + W) * ldx + c]));
    m = fmaxf(m, bf2f(X[(base + W + 1) * ldx + c]));
    Y[e] = f2bf(m);
  }
}

hipError_t pool_fwd(const uint16_t* X, int64_t ldx, int C, int B, int H, int W, uint16_t* Y,
                    hipStream_t st) {
  const int64_t total = (int64_t)B * (H / 2) * (W / 2) * C;
  hipLaunchKernelGGL(k_pool_fwd, dim3(blocks_for(total)), dim3(256), 0, st, X, ldx, C, B, H, W,
                     Y);
  return hipGetLastError();
}

__global__ void k_pool_bwd(const uint16_t* X, int64_t ldx, const uint16_t* dY, int C, int B,
                           int H, int W, uint16_t* dX) {
  const int Ho = H / 2, Wo = W / 2;
  const int64_t total = (int64_t)B * Ho * Wo * C;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const int64_t p = e / C;
    const int x = (int)(p % Wo);
    const int y = (int)((p / Wo) % Ho);
    const int64_t b = p / ((int64_t)Wo * Ho);
    const int64_t base = (b * H + 2 * y) * W + 2 * x;
    const int64_t cand[4] = {base, base + 1, base + W, base + W + 1};
    int arg = 0;
    float m = bf2f(X[cand[0] * ldx + c]);
#pragma unroll
    for (int q = 1; q < 4; ++q) {
      const float v = bf2f(X[cand[q] * ldx + c]);
      if (v > m) {
        m = v;
        arg = q;
      }
    }
    uint16_t* d = &dX[cand[arg] * ldx + c];
    *d = f2bf(bf2f(*d) + bf2f(dY[e]));
  }
}

hipError_t pool_bwd(const uint16_t* X, int64_t ldx, const uint16_t* dY, int C, int B, int H,
                    int W, uint16_t* dX, hipStream_t st) {
  const int64_t total = (int64_t)B * (H / 2) * (W / 2) * C;
  hipLaunchKernelGGL(k_pool_bwd, dim3(blocks_for(total)), dim3(256), 0, st, X, ldx, dY, C, B, H,
                     W, dX);
  return hipGetLastError();
}

// Space-to-depth, the adjoint of the transposed convolution's stores: one
// element, or eight (C and ldy multiples of 8, 16-byte aligned), per (low-res
// pixel, a, c, channel group).
template <int V>
__global__ void k_s2d(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int C, int B,
                      int H, int W, int64_t ldy) {
  const int CV = C / V;
  const int64_t total = (int64_t)B * H * W * 4 * CV;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int ch = (int)(e % CV) * V;
    const int64_t q = e / CV;
    const int ac = (int)(q & 3);
    const uint32_t p = (uint32_t)(q >> 2);  // < 2^28 pixels
    const uint32_t yb = p / W, x = p - yb * W;
    const int64_t py = (int64_t)(2 * yb + (ac >> 1)) * (2 * W) + 2 * x + (ac & 1);
    if (V == 8)
      *reinterpret_cast<u4v*>(dst + e * 8) = *reinterpret_cast<const u4v*>(src + py * ldy + ch);
    else
      dst[e] = src[py * ldy + ch];
  }
}

hipError_t s2d(const uint16_t* Y, int64_t ldy, int C, int B, int H, int W, uint16_t* S,
               hipStream_t st) {
  const int64_t total = (int64_t)B * H * W * 4 * C;
  if (C % 8 == 0 && ldy % 8 == 0 && (((uintptr_t)Y | (uintptr_t)S) & 15) == 0)
    hipLaunchKernelGGL(k_s2d<8>, dim3(blocks_for(total / 8)), dim3(256), 0, st, Y, S, C, B, H, W,
                       ldy);
  else
    hipLaunchKernelGGL(k_s2d<1>, dim3(blocks_for(total)), dim3(256), 0, st, Y, S, C, B, H, W, ldy);
  return hipGetLastError();
}

__global__ void k_relu_bwd(uint16_t* dY, int64_t lddy, const uint16_t* Y, int64_t ldy, int C,
                           int64_t P) {
  const int64_t total = P * C;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const int64_t p = e / C;
    if (!(bf2f(Y[p * ldy + c]) > 0.f)) dY[p * lddy + c] = 0;
  }
}

hipError_t relu_bwd(uint16_t* dY, int64_t lddy, const uint16_t* Y, int64_t ldy, int C, int64_t P,
                    hipStream_t st) {
  hipLaunchKernelGGL(k_relu_bwd, dim3(blocks_for(P * C)), dim3(256), 0, st, dY, lddy, Y, ldy, C,
                     P);
  return hipGetLastError();
}

// Column sums of P rows: block (cx, r) takes channels 64 cx .. +63 of rows r
// 32 + .., its thread eight channels (one 16-byte load per row where the rows
// allow it) of every 32 nblk-th row; combined in LDS.
__global__ __launch_bounds__(256) void k_colsum(const uint16_t* __restrict__ dY, int64_t ld, int C,
                                                int64_t P, float* __restrict__ part) {
  __shared__ float red[32][64];
  const int c8 = 8 * (threadIdx.x & 7), r = threadIdx.x >> 3;
  const int c = blockIdx.x * 64 + c8;
  const bool vec = c + 8 <= C && ld % 8 == 0 && ((uintptr_t)dY & 15) == 0;
  float s[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = 0.f;
  if (vec) {
#pragma unroll 4
    for (int64_t p = (int64_t)blockIdx.y * 32 + r; p < P; p += (int64_t)gridDim.y * 32) {
      const u4v v = *reinterpret_cast<const u4v*>(dY + p * ld + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[2 * e] += __uint_as_float(v[e] << 16);
        s[2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u);
      }
    }
  } else if (c < C) {
    for (int64_t p = (int64_t)blockIdx.y * 32 + r; p < P; p += (int64_t)gridDim.y * 32)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (c + e < C) s[e] += bf2f(dY[p * ld + c + e]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[r][c8 + e] = s[e];
  __syncthreads();
  if (threadIdx.x < 64 && blockIdx.x * 64 + threadIdx.x < C) {
    float v = 0.f;
#pragma unroll 8
    for (int k = 0; k < 32; ++k) v += red[k][threadIdx.x];
    part[(int64_t)blockIdx.y * C + blockIdx.x * 64 + threadIdx.x] = v;
  }
}

hipError_t colsum(const uint16_t* dY, int64_t ld, int C, int64_t P, float* part, int nblk,
                  float* db, hipStream_t st) {
  hipLaunchKernelGGL(k_colsum, dim3((C + 63) / 64, nblk), dim3(256), 0, st, dY, ld, C, P, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return sum_slices(part, nblk, C, db, st);
}

// Rows of Wb and Wt are padded to multiples of 32 (the padding is zeroed when
// the model is made).
__global__ void k_weight_copies(const float* __restrict__ W, int Cin, int Cout, int K,
                                uint16_t* __restrict__ Wb, uint16_t* __restrict__ Wt) {
  const int KK = K * K;
  const int64_t total = (int64_t)KK * Cin * Cout;
  const int64_t ldb = conv_row(KK * Cin), ldt = conv_row(KK * Cout);
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int co = (int)(e % Cout);
    const int64_t q = e / Cout;
    const int ci = (int)(q % Cin);
    const int kk = (int)(q / Cin);
    const uint16_t v = f2bf(W[e]);
    Wb[co * ldb + q] = v;
    const int kh = kk / K, kw = kk % K;
    const int kf = (K - 1 - kh) * K + (K - 1 - kw);
    Wt[ci * ldt + (int64_t)kf * Cout + co] = v;
  }
}

hipError_t weight_copies(const float* W, int Cin, int Cout, int K, uint16_t* Wb, uint16_t* Wt,
                         hipStream_t st) {
  const int64_t total = (int64_t)K * K * Cin * Cout;
  hipLaunchKernelGGL(k_weight_copies, dim3(blocks_for(total)), dim3(256), 0, st, W, Cin, Cout, K,
                     Wb, Wt);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_masked_loss(const float* pred, int nt,
                                                     const LabelRec* lab, int n, float inv_n,
                                                     uint16_t* dpred, double* part) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const LabelRec L = lab[i];
    const int64_t at = (int64_t)L.pix * nt + L.t;
    const float d = pred[at] - L.logR;
    dpred[at] = f2bf(2.f * d * inv_n);
    s += (double)d * (double)d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

hipError_t masked_loss(const float* pred, int nt, const LabelRec* lab, int n, float inv_n,
                       uint16_t* dpred, double* part, int nblk, hipStream_t st) {
  hipLaunchKernelGGL(k_masked_loss, dim3(nblk), dim3(256), 0, st, pred, nt, lab, n, inv_n, dpred,
                     part);
  return hipGetLastError();
}

__global__ void k_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, float bc1, float bc2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  }
}

hipError_t adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                float b2, float eps, float bc1, float bc2, hipStream_t st) {
  hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2,
                     eps, bc1, bc2);
  return hipGetLastError();
}

__global__ void k_fill16(uint16_t* a, int64_t n, uint16_t val) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = val;
}

hipError_t fill16(uint16_t* a, int64_t n, uint16_t val, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill16, dim3(blocks_for(n)), dim3(256), 0, st, a, n, val);
  return hipGetLastError();
}

__global__ void k_predict_out(const float* pred, const uint8_t* padm, int B, int nt, int H, int W,
                              double* R) {
  const int64_t HW = (int64_t)H * W;
  const int64_t total = (int64_t)B * nt * HW;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t pix = e % HW;
    const int t = (int)((e / HW) % nt);
    const int64_t b = e / (HW * nt);
    R[e] = padm[b * HW + pix] && t == 0 ? 0.0 : exp((double)pred[(b * HW + pix) * nt + t]);
  }
}

hipError_t predict_out(const float* pred, const uint8_t* padm, int B, int nt, int H, int W,
                       double* R, hipStream_t st) {
  const int64_t total = (int64_t)B * nt * H * W;
  hipLaunchKernelGGL(k_predict_out, dim3(blocks_for(total)), dim3(256), 0, st, pred, padm, B, nt,
                     H, W, R);
  return hipGetLastError();
}

}  // namespace reffsg
