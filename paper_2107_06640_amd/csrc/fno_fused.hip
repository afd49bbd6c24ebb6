// Fused kernels of the spectral neural operator (include/fno.h): each stage of
// a layer reads its activations once and writes its result once, where a chain
// of general products (fno.hip) writes and re-reads every intermediate.
//
// All products are v_mfma_f32_16x16x32_bf16 with the operands rounded to BF16
// and FP32 accumulation, over the same 32-wide K steps in the same order as
// k_gemm, and sums of two products add the finished FP32 accumulators, so the
// activations and their gradients equal those of the general path bit for bit
// (a different rounding anywhere would flip BF16 roundings further down the
// network). Only the weight gradients, sums over all points that nothing
// rounds again, are summed in another order.
//
// The stages over the grid move little but their activations, at half to three quarters of the
// rate of a large copy (4.9 TB/s); what keeps them below it is the latency of a work-group's phases
// (loads, products, exchange through LDS, stores). The projection is bound by the erf and exp of
// GELU. Measured on 64 samples of a 64 x 64 x 32 grid, width 32, 12 modes, hidden width 128 (an
// activation is 1.07 GB), average per call in a training step: k_idft_yt 854 us (two or
// three activations, 2.5-3.8 TB/s), k_layer_bwd 1039 (three, 3.1), k_dft_ty 315 (one,
// 3.4), k_dft_x 100, k_mix 108, k_mix_grad 94, k_pointwise 273, k_head 575 and k_head_bwd
// 1944 (GELU and its derivative of 128 hidden values a point). The step takes 18.8 ms, with the general
// products 160.5 ms; one sample's inference 0.35 and 2.15 ms.
//
// Fragment conventions (lane l, g = l / 16, c = l % 16): A holds row c, K
// entries 8g..8g+7; B holds column c, the same K entries; the result holds
// rows 4g..4g+3 of column c.
//
// Channel-planar activations [channel][point]: a wavefront takes 64 points as
// four 16-column products whose column c of product u is point 4c + u, so a
// lane's four columns are four consecutive points, one 16-byte access.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "../../include/fno.h"
#include "lds_limit.hpp"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16;

// shapes the kernels are compiled for (register tiles and LDS images)
constexpr int kMaxW = 48, kMaxH = 256, kMaxModes = 16, kMaxT = 64, kMaxXY = 128;
constexpr int kLds = 160 * 1024;

__host__ __device__ constexpr int up(int x, int m) { return (x + m - 1) / m * m; }

__device__ __forceinline__ f4 mfma(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f4 zero4() { return f4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ bf8 pack8(f8 x) { return __builtin_convertvector(x, bf8); }
__device__ __forceinline__ bf4 pack4(f4 x) { return __builtin_convertvector(x, bf4); }
__device__ __forceinline__ u16 bits(float x) { return __builtin_bit_cast(u16, (__bf16)x); }
__device__ __forceinline__ float rounded(float x) { return (float)(__bf16)x; }
// eight consecutive BF16 values of an LDS row (16-byte aligned)
__device__ __forceinline__ bf8 lds8(const u16* p) { return *reinterpret_cast<const bf8*>(p); }
__device__ __forceinline__ void put4(u16* p, f4 x) { *reinterpret_cast<bf4*>(p) = pack4(x); }

// orders a wavefront's LDS writes before the reads of its other lanes
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// Mask of a fragment's eight K entries 8g.. of the last 32, of which n are real: the others
// meet zeros, but 0 x inf would not be zero where an activation is infinite.
typedef unsigned u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u4 last_mask(int n, int g) {
  u4 m;
#pragma unroll
  for (int j = 0; j < 4; ++j) m[j] = (8 * g + 2 * j < n ? 0xffffu : 0u) | (8 * g + 2 * j + 1 < n ? 0xffff0000u : 0u);
  return m;
}
__device__ __forceinline__ bf8 masked(bf8 x, u4 m) { return __builtin_bit_cast(bf8, __builtin_bit_cast(u4, x) & m); }

// four consecutive values from i on, zero from n on; V4: p is 16-byte aligned and n a multiple of 4
template <bool V4>
__device__ __forceinline__ f4 load4(const float* p, int64_t i, int64_t n) {
  if constexpr (V4) {
    return i < n ? *reinterpret_cast<const f4*>(p + i) : zero4();
  } else {
    f4 r;
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = i + u < n ? p[i + u] : 0.0f;
    return r;
  }
}
template <bool V4>
__device__ __forceinline__ void store4(float* p, int64_t i, int64_t n, f4 x) {
  if constexpr (V4) {
    if (i < n) *reinterpret_cast<f4*>(p + i) = x;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u < n) p[i + u] = x[u];
  }
}

// dst[r][k] = BF16 of src(r, k) = src[r * sr + k * sk], zero outside rows x cols, for a
// prows x pcols image (pcols a multiple of 8) with leading dimension ld. A thread moves eight
// K entries at a time, so that their loads are in flight together; consecutive threads walk
// the unit-stride index.
__device__ __forceinline__ void stage(u16* dst, const float* src, int64_t sr, int64_t sk, int rows, int cols,
                                      int prows, int pcols, int ld, int tid, int nt) {
  const int k8s = pcols / 8;
  for (int i = tid; i < prows * k8s; i += nt) {
    int r, k;
    if (sk == 1) { r = i / k8s; k = 8 * (i - r * k8s); } else { k = i / prows; r = i - k * prows; k *= 8; }
    f8 x;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = (r < rows && k + j < cols) ? src[r * sr + (k + j) * sk] : 0.0f;
    *reinterpret_cast<bf8*>(dst + r * ld + k) = pack8(x);
  }
}

// B fragments of 64 points of an activation x[ci][n], K entries 32 kc + 8g..: four column sets
template <bool V4>
__device__ __forceinline__ void point_frags(const float* x, int64_t p, int64_t n, int cin, int kc, int g, bf8 (&b)[4]) {
  f4 v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int ci = 32 * kc + 8 * g + j;
    v[j] = ci < cin ? load4<V4>(x + (int64_t)ci * n, p, n) : zero4();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) b[u] = pack8(f8{v[0][u], v[1][u], v[2][u], v[3][u], v[4][u], v[5][u], v[6][u], v[7][u]});
}

// ---------------------------------------------------------------------------
// z[o][p] = sum_i Wm[o][i] x[i][p] + bias[o]: the network's lift. Bound by the
// write of z; one pass instead of a product, then a pass for the bias.
template <int MT, bool V4>
__global__ __launch_bounds__(256) void k_pointwise(int64_t n, int cout, int cin, const float* Wm, const float* x,
                                                   const float* bias, float* z) {
  constexpr int LD = 64 + 8;
  __shared__ __align__(16) u16 sW[16 * MT * LD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int KC = (cin + 31) / 32;
  stage(sW, Wm, cin, 1, cout, cin, 16 * MT, 32 * KC, LD, tid, 256);
  __syncthreads();
  const int64_t tiles = (n + 63) / 64;
  for (int64_t t = (int64_t)blockIdx.x * 4 + w; t < tiles; t += (int64_t)gridDim.x * 4) {
    const int64_t p = t * 64 + 4 * c;
    f4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[mt][u] = zero4();
    for (int kc = 0; kc < KC; ++kc) {
      bf8 b[4];
      point_frags<V4>(x, p, n, cin, kc, g, b);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf8 a = lds8(sW + (16 * mt + c) * LD + 32 * kc + 8 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[mt][u] = mfma(a, b[u], acc[mt][u]);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int o = 16 * mt + 4 * g + v;
        if (o >= cout) continue;
        const float bb = bias[o];
        store4<V4>(z + (int64_t)o * n, p, n, f4{acc[mt][0][v] + bb, acc[mt][1][v] + bb, acc[mt][2][v] + bb, acc[mt][3][v] + bb});
      }
  }
}

// ---------------------------------------------------------------------------
// Projection y = Q2 gelu(Q1 v + q1) + q2 at 64 points per work-group: each
// wavefront forms 32 hidden rows (HC per wavefront) from its fragments of v,
// applies the activation in registers and leaves it in LDS as the K entries of
// the second product, of which wavefront w takes points 16w..16w+15. Nothing
// of the H x n hidden activation reaches memory (it was written and read five
// times); bound by the erf of the activation (VALU) and the read of v.
template <int KC, int HC, bool V4>
__global__ __launch_bounds__(256) void k_head(int64_t n, int W, int H, const float* Q1, const float* q1,
                                              const float* Q2, const float* q2, const float* v, float* y) {
  constexpr int LD = 128 * HC + 8;
  extern __shared__ __align__(16) u16 sm[];  // two buffers of gelu(h)[point][h]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int chunks = (H + 31) / 32;
  bf8 a1[HC][2][KC];
  float b1[HC][2][4];
#pragma unroll
  for (int h = 0; h < HC; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = 32 * (w + 4 * h) + 16 * i;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        f8 x;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 32 * kc + 8 * g + j;
          x[j] = (row + c < H && k < W) ? Q1[(row + c) * W + k] : 0.0f;
        }
        a1[h][i][kc] = pack8(x);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) b1[h][i][r] = row + 4 * g + r < H ? q1[row + 4 * g + r] : 0.0f;
    }
  bf8 a2[4 * HC];
#pragma unroll
  for (int k = 0; k < 4 * HC; ++k) {
    f8 x;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = (c == 0 && 32 * k + 8 * g + j < H) ? Q2[32 * k + 8 * g + j] : 0.0f;
    a2[k] = pack8(x);
  }
  const float b2 = q2[0];
  const u4 last = last_mask(H - 32 * (chunks - 1), g);
  const int64_t tiles = (n + 63) / 64;
  int buf = 0;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x, buf ^= 1) {
    const int64_t p0 = t * 64;
    bf8 b[KC][4];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) point_frags<V4>(v, p0 + 4 * c, n, W, kc, g, b[kc]);
    u16* G = sm + buf * 64 * LD;
#pragma unroll
    for (int h = 0; h < HC; ++h) {
      if (w + 4 * h >= chunks) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          f4 acc = zero4();
#pragma unroll
          for (int kc = 0; kc < KC; ++kc) acc = mfma(a1[h][i][kc], b[kc][u], acc);
          f4 x;
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = gelu(acc[r] + b1[h][i][r]);
          put4(G + (4 * c + u) * LD + 32 * (w + 4 * h) + 16 * i + 4 * g, x);
        }
    }
    __syncthreads();  // one barrier per tile: the other buffer is written next
    f4 acc = zero4();
#pragma unroll
    for (int k = 0; k < 4 * HC; ++k)
      if (k < chunks) {
        bf8 x = lds8(G + (16 * w + c) * LD + 32 * k + 8 * g);
        if (k == chunks - 1) x = masked(x, last);
        acc = mfma(a2[k], x, acc);
      }
    const int64_t p = p0 + 16 * w + c;
    if (g == 0 && p < n) y[p] = acc[0] + b2;
  }
}

// Gradients of the projection for dy[n]: the hidden activation is formed again
// from v (cheaper than keeping it), dh = Q2^T dy gelu'(h), dv = Q1^T dh, and
// dQ1, dq1, dQ2 summed over the points in registers and added to memory once
// per work-group (cleared before).
template <int KC, int HC, bool V4>
__global__ __launch_bounds__(256, KC * HC == 1 ? 2 : 1) void k_head_bwd(int64_t n, int W, int H, const float* Q1, const float* q1,
                                                  const float* Q2, const float* v, const float* dy, float* dv,
                                                  float* dQ1, float* dq1, float* dQ2) {
  constexpr int LD = 128 * HC + 8, LP = 64 + 8, WT = 2 * KC;
  extern __shared__ __align__(16) unsigned char smem[];
  u16* sD = reinterpret_cast<u16*>(smem);  // dh[point][h]
  u16* sT = sD + 64 * LD;                  // dh[h][point]
  u16* sV = sT + 128 * HC * LP;            // v[ci][point]
  u16* sQ = sV + 32 * KC * LP;             // Q1^T[ci][h]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int chunks = (H + 31) / 32;
  stage(sQ, Q1, 1, W, W, H, 32 * KC, 128 * HC, LD, tid, 256);
  const u4 last = last_mask(H - 32 * (chunks - 1), g);
  bf8 a1[HC][2][KC];
  float b1[HC][2][4], q2b[HC][2][4], s1[HC][2][4], s2[HC][2][4];
  f4 dw[HC][2][WT];
#pragma unroll
  for (int h = 0; h < HC; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = 32 * (w + 4 * h) + 16 * i;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        f8 x;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 32 * kc + 8 * g + j;
          x[j] = (row + c < H && k < W) ? Q1[(row + c) * W + k] : 0.0f;
        }
        a1[h][i][kc] = pack8(x);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int hr = row + 4 * g + r;
        b1[h][i][r] = hr < H ? q1[hr] : 0.0f;
        q2b[h][i][r] = hr < H ? rounded(Q2[hr]) : 0.0f;
        s1[h][i][r] = s2[h][i][r] = 0.0f;
      }
#pragma unroll
      for (int nt = 0; nt < WT; ++nt) dw[h][i][nt] = zero4();
    }
  __syncthreads();
  const int64_t tiles = (n + 63) / 64;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t p0 = t * 64, p = p0 + 4 * c;
    f4 d4 = load4<V4>(dy, p, n);
#pragma unroll
    for (int u = 0; u < 4; ++u) d4[u] = rounded(d4[u]);
    bf8 b[KC][4];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) point_frags<V4>(v, p, n, W, kc, g, b[kc]);
    // v[ci][point], a quarter of the rows per wavefront
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if ((j >> 1) == w)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const __bf16 x = b[kc][u][j];
            sV[(32 * kc + 8 * g + j) * LP + 4 * c + u] = __builtin_bit_cast(u16, x);
          }
#pragma unroll
    for (int h = 0; h < HC; ++h) {
      if (w + 4 * h >= chunks) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = 32 * (w + 4 * h) + 16 * i + 4 * g;
        f4 dh[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          f4 acc = zero4();
#pragma unroll
          for (int kc = 0; kc < KC; ++kc) acc = mfma(a1[h][i][kc], b[kc][u], acc);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x = acc[r] + b1[h][i][r];
            const float d = q2b[h][i][r] * d4[u] * gelu_d(x);
            dh[u][r] = d;
            s1[h][i][r] += d;
            s2[h][i][r] += d4[u] * rounded(gelu(x));
          }
          put4(sD + (4 * c + u) * LD + row, dh[u]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) put4(sT + (row + r) * LP + 4 * c, f4{dh[0][r], dh[1][r], dh[2][r], dh[3][r]});
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < HC; ++h) {
      if (w + 4 * h >= chunks) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) {
          const bf8 a = lds8(sT + (32 * (w + 4 * h) + 16 * i + c) * LP + 32 * kp + 8 * g);
#pragma unroll
          for (int nt = 0; nt < WT; ++nt)
            dw[h][i][nt] = mfma(a, lds8(sV + (16 * nt + c) * LP + 32 * kp + 8 * g), dw[h][i][nt]);
        }
    }
    const int64_t q = p0 + 16 * w + c;
#pragma unroll
    for (int mt = 0; mt < WT; ++mt) {
      f4 acc = zero4();
      for (int k = 0; k < chunks - 1; ++k)
        acc = mfma(lds8(sQ + (16 * mt + c) * LD + 32 * k + 8 * g), lds8(sD + (16 * w + c) * LD + 32 * k + 8 * g), acc);
      const int k = 32 * (chunks - 1) + 8 * g;
      acc = mfma(lds8(sQ + (16 * mt + c) * LD + k), masked(lds8(sD + (16 * w + c) * LD + k), last), acc);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (16 * mt + 4 * g + r < W && q < n) dv[(int64_t)(16 * mt + 4 * g + r) * n + q] = acc[r];
    }
    __syncthreads();
  }
#pragma unroll
  for (int h = 0; h < HC; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float x = s1[h][i][r], z = s2[h][i][r];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
          x += __shfl_xor(x, o, 64);
          z += __shfl_xor(z, o, 64);
        }
        const int hr = 32 * (w + 4 * h) + 16 * i + 4 * g + r;
        if (hr >= H) continue;
        if (c == 0) {
          atomicAdd(dq1 + hr, x);
          atomicAdd(dQ2 + hr, z);
        }
#pragma unroll
        for (int nt = 0; nt < WT; ++nt)
          if (16 * nt + c < W) atomicAdd(dQ1 + hr * W + 16 * nt + c, dw[h][i][nt][r]);
      }
}

// ---------------------------------------------------------------------------
// Backward of a pointwise product z = Wm x (+ activation): dz = da gelu'(z)
// (ACT; otherwise dz is da), dW = sum_p dz x^T and db = sum_p dz, summed in
// registers, then over the work-group, and added to memory (cleared before).
// One pass over z, da and x; bound by these reads and the write of dz.
template <int MT, int NT, bool ACT, bool V4>
__global__ __launch_bounds__(256) void k_layer_bwd(int64_t n, int cout, int cin, const float* z, const float* da,
                                                   const float* x, float* dz, float* dW, float* db) {
  constexpr int LP = 64 + 8;
  __shared__ __align__(16) u16 sD[4][16 * MT * LP], sX[4][16 * NT * LP];
  __shared__ float sR[16 * MT][16 * NT + 1];  // the work-group's dW and, last column, db
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  u16 *D = sD[w], *Xs = sX[w];
  for (int i = tid; i < 16 * MT * (16 * NT + 1); i += 256) (&sR[0][0])[i] = 0.0f;
  f4 acc[MT][NT];
  float s[4 * MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = zero4();
#pragma unroll
  for (int i = 0; i < 4 * MT; ++i) s[i] = 0.0f;
  const int64_t tiles = (n + 63) / 64;
  for (int64_t t = (int64_t)blockIdx.x * 4 + w; t < tiles; t += (int64_t)gridDim.x * 4) {
    const int64_t p = t * 64 + 4 * c;
    f4 d[4 * MT], xx[4 * NT];
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i) {
      const int o = 4 * i + g;
      d[i] = o < cout ? load4<V4>(da + (int64_t)o * n, p, n) : zero4();
    }
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) {
      const int o = 4 * i + g;
      xx[i] = o < cin ? load4<V4>(x + (int64_t)o * n, p, n) : zero4();
    }
    if constexpr (ACT) {
#pragma unroll
      for (int i = 0; i < 4 * MT; ++i) {
        const int o = 4 * i + g;
        if (o >= cout) continue;
        const f4 zz = load4<V4>(z + (int64_t)o * n, p, n);
#pragma unroll
        for (int u = 0; u < 4; ++u) d[i][u] *= gelu_d(zz[u]);
        store4<V4>(dz + (int64_t)o * n, p, n, d[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i) {
      s[i] += (d[i][0] + d[i][1]) + (d[i][2] + d[i][3]);
      put4(D + (4 * i + g) * LP + 4 * c, d[i]);
    }
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) put4(Xs + (4 * i + g) * LP + 4 * c, xx[i]);
    wave_sync();
#pragma unroll
    for (int kp = 0; kp < 2; ++kp) {
      bf8 b[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) b[j] = lds8(Xs + (16 * j + c) * LP + 32 * kp + 8 * g);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const bf8 a = lds8(D + (16 * i + c) * LP + 32 * kp + 8 * g);
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = mfma(a, b[j], acc[i][j]);
      }
    }
    wave_sync();
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4 * MT; ++i) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) s[i] += __shfl_xor(s[i], o, 64);
    if (c == 0) atomicAdd(&sR[4 * i + g][16 * NT], s[i]);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) atomicAdd(&sR[16 * i + 4 * g + r][16 * j + c], acc[i][j][r]);
  __syncthreads();
  for (int i = tid; i < cout * (cin + 1); i += 256) {
    const int o = i / (cin + 1), k = i - o * (cin + 1);
    if (k < cin) atomicAdd(dW + o * cin + k, sR[o][k]);
    else atomicAdd(db + o, sR[o][16 * NT]);
  }
}

// ---------------------------------------------------------------------------
// Truncated transforms along t and y of every slice v[Y][T]:
//   U[y][(p, kt)] = sum_t v[y][t] Bt(t, (p, kt)),
//   out[r][kt] = sum_y F1[r][y] U[y][(1, kt)] + sum_y F0[r][y] U[y][(0, kt)].
// A wavefront takes a slice; its U goes from the first product's result to the
// second's operand through the wavefront's own LDS rows (BF16, as the operand
// is), so the 2m x Y intermediate never reaches memory. Bound by the read of v.
struct TyArgs {
  int64_t slices;
  int Y, T, m;
  const float* v;
  const float *Bt, *F0, *F1;
  int64_t sBk, sBn, sFm, sFk;
  float* out;
};

struct TyLds {
  int Yp, Tp, Rp, Np, ldF, ldB, offB, offU, wave, total;  // in BF16 values
  __host__ __device__ TyLds(int Y, int T, int m) {
    Yp = up(Y, 32);
    Tp = up(T, 32);
    Rp = up(4 * m, 16);
    Np = up(2 * m, 16);
    ldF = Yp + 8;
    ldB = Tp + 8;
    offB = 2 * Rp * ldF;
    offU = offB + Np * ldB;
    wave = (Np + 16) * ldF;  // rows p m + 0..15 are read for both parts
    total = offU + 4 * wave;
  }
};

template <int TC, bool V4>
__global__ __launch_bounds__(256) void k_dft_ty(TyArgs a) {
  extern __shared__ __align__(16) u16 sm[];
  const TyLds L(a.Y, a.T, a.m);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int m = a.m, m2 = 2 * m, Y = a.Y, T = a.T;
  stage(sm, a.F0, a.sFm, a.sFk, 4 * m, Y, L.Rp, L.Yp, L.ldF, tid, 256);
  stage(sm + L.Rp * L.ldF, a.F1, a.sFm, a.sFk, 4 * m, Y, L.Rp, L.Yp, L.ldF, tid, 256);
  stage(sm + L.offB, a.Bt, a.sBn, a.sBk, m2, T, L.Np, L.Tp, L.ldB, tid, 256);
  u16* U = sm + L.offU + w * L.wave;
  for (int i = lane; i < L.wave; i += 64) U[i] = 0;
  __syncthreads();
  const int MT = (Y + 15) / 16, NT = L.Np / 16, RT = L.Rp / 16, YC = L.Yp / 32;
  for (int64_t s = (int64_t)blockIdx.x * 4 + w; s < a.slices; s += (int64_t)gridDim.x * 4) {
    const float* v = a.v + s * Y * T;
#pragma unroll 4
    for (int mt = 0; mt < MT; ++mt) {
      const int y = 16 * mt + c;
      bf8 av[TC];
#pragma unroll
      for (int kc = 0; kc < TC; ++kc) {
        const int t = 32 * kc + 8 * g;
        const float* row = v + (y < Y ? y : 0) * T;
        const f4 lo = load4<V4>(row, t, y < Y ? T : 0), hi = load4<V4>(row, t + 4, y < Y ? T : 0);
        av[kc] = pack8(f8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
      }
      for (int nt = 0; nt < NT; ++nt) {
        f4 acc = zero4();
#pragma unroll
        for (int kc = 0; kc < TC; ++kc) acc = mfma(av[kc], lds8(sm + L.offB + (16 * nt + c) * L.ldB + 32 * kc + 8 * g), acc);
        put4(U + (16 * nt + c) * L.ldF + 16 * mt + 4 * g, acc);
      }
    }
    wave_sync();
    float* out = a.out + s * 4 * m * m;
    for (int rt = 0; rt < RT; ++rt) {
      f4 a0 = zero4(), a1 = zero4();
      for (int kc = 0; kc < YC; ++kc) {
        const int k = 32 * kc + 8 * g, ra = (16 * rt + c) * L.ldF + k;
        a0 = mfma(lds8(sm + ra), lds8(U + c * L.ldF + k), a0);
        a1 = mfma(lds8(sm + L.Rp * L.ldF + ra), lds8(U + (m + c) * L.ldF + k), a1);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * g + r;
        if (row < 4 * m && c < m) out[row * m + c] = a1[r] + a0[r];
      }
    }
    wave_sync();
  }
}

// ---------------------------------------------------------------------------
// Transforms along x: out[b](q, r, j) = sum over the parts p of
// sum_k A(p, q)[r][k] in[b][k][p][j], j < inner. Forward: two parts (real and
// imaginary), one q; inverse: one part whose K holds both, two q (the real and
// the imaginary result). A work-group takes 32 columns j of a batch entry.
struct XArgs {
  int64_t batch;
  int M, K, inner, parts, nq;   // rows per q, K per part
  const float *A0, *A1;         // the matrices of part (or q) 0 and 1
  int64_t sAm, sAk;
  const float* in;              // [batch][K][parts][inner]
  float* out;                   // [batch]: element (q, r, j) at q sq + r sr + j
  int64_t sob, sq, sr;
};

constexpr int kXCols = 32;

__global__ __launch_bounds__(256) void k_dft_x(XArgs a) {
  extern __shared__ __align__(16) u16 sm[];
  const int Kp = up(a.K, 32), ld = Kp + 8, Mp = up(a.M, 16), P = a.parts, mats = a.parts * a.nq;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  for (int i = 0; i < mats; ++i) stage(sm + i * Mp * ld, i ? a.A1 : a.A0, a.sAm, a.sAk, a.M, a.K, Mp, Kp, ld, tid, 256);
  u16* sB = sm + mats * Mp * ld;  // [part][column][k]
  for (int i = tid; i < P * kXCols * ld; i += 256) sB[i] = 0;
  const int chunks = (a.inner + kXCols - 1) / kXCols, RT = Mp / 16 * a.nq;
  const int64_t tasks = a.batch * chunks;
  for (int64_t t = blockIdx.x; t < tasks; t += gridDim.x) {
    const int64_t b = t / chunks;
    const int j0 = int(t - b * chunks) * kXCols;
    const float* in = a.in + b * a.K * P * a.inner + j0;
    __syncthreads();
    // a thread moves two K entries of two columns (inner is even: aligned 8-byte loads), four such
    // blocks in flight
    const int blocks = (a.K + 1) / 2 * P * (kXCols / 2);
    for (int i0 = tid; i0 < blocks; i0 += 4 * 256) {
      f2 x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 256 * u, jj = 2 * (i % (kXCols / 2)), kp = i / (kXCols / 2), p = kp % P, k = 2 * (kp / P);
        const bool ok = i < blocks && j0 + jj < a.inner;
        const float* q = in + (int64_t)(k * P + p) * a.inner + jj;
        x[u] = ok ? *reinterpret_cast<const f2*>(q) : f2{0.f, 0.f};
        y[u] = ok && k + 1 < a.K ? *reinterpret_cast<const f2*>(q + (int64_t)P * a.inner) : f2{0.f, 0.f};
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 256 * u, jj = 2 * (i % (kXCols / 2)), kp = i / (kXCols / 2), p = kp % P, k = 2 * (kp / P);
        if (i >= blocks) continue;
        *reinterpret_cast<bf2*>(sB + (p * kXCols + jj) * ld + k) = __builtin_convertvector(f2{x[u][0], y[u][0]}, bf2);
        *reinterpret_cast<bf2*>(sB + (p * kXCols + jj + 1) * ld + k) = __builtin_convertvector(f2{x[u][1], y[u][1]}, bf2);
      }
    }
    __syncthreads();
    for (int i = w; i < RT * (kXCols / 16); i += 4) {
      const int nt = i % (kXCols / 16), rq = i / (kXCols / 16), q = rq / (Mp / 16), rt = rq - q * (Mp / 16);
      f4 acc[2] = {zero4(), zero4()};
      for (int p = 0; p < P; ++p)
        for (int kc = 0; kc < Kp / 32; ++kc) {
          const bf8 x = lds8(sm + ((p + q) * Mp + 16 * rt + c) * ld + 32 * kc + 8 * g);
          const bf8 y = lds8(sB + (p * kXCols + 16 * nt + c) * ld + 32 * kc + 8 * g);
          if (p == 0) acc[0] = mfma(x, y, acc[0]);
          else acc[1] = mfma(x, y, acc[1]);
        }
      const int j = j0 + 16 * nt + c;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * g + r;
        if (row < a.M && j < a.inner) a.out[b * a.sob + q * a.sq + row * a.sr + j] = P == 2 ? acc[1][r] + acc[0][r] : acc[0][r];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Per-mode complex channel mixing: with in and out [c][b][re, im][mode] and
// R [re, im][mode](i, o), for each mode
//   out_re = in_re R_re + s_re (in_im R_im),  out_im = in_im R_re + s_im (in_re R_im).
// A work-group takes 16 consecutive modes, so that the strided activations move
// in 64-byte runs through LDS (a batched product over modes gathers them four
// bytes at a time); a wavefront keeps the R fragments of its two modes in
// registers over all batch tiles. Bound by the read of R at small batches, by
// the activations at large ones.
constexpr int kMixModes = 16, kMixWaves = 8;

template <int NT>
__global__ __launch_bounds__(64 * kMixWaves) void k_mix(int B, int W, int64_t nm, const float* in, const float* R,
                                                        int64_t sRi, int64_t sRo, float s_re, float s_im, float* out) {
  constexpr int KC = (NT + 1) / 2, LD = 32 * KC + 8, NTH = 64 * kMixWaves, LO = kMixModes + 1;
  extern __shared__ __align__(16) unsigned char smem[];
  u16* sI = reinterpret_cast<u16*>(smem);      // [re, im][mode][b][ci]
  float* sO = reinterpret_cast<float*>(smem);  // [re, im][co][b][mode], in the same place
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int64_t m0 = (int64_t)blockIdx.x * kMixModes;
  bf8 r[2][2][NT][KC];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t mode = m0 + 2 * w + i < nm ? m0 + 2 * w + i : nm - 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float* Rm = R + (q * nm + mode) * W * W;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
          f8 x;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int k = 32 * kc + 8 * g + j, o = 16 * nt + c;
            x[j] = (k < W && o < W) ? Rm[k * sRi + o * sRo] : 0.0f;
          }
          r[i][q][nt][kc] = pack8(x);
        }
    }
  }
  const int64_t sb = 2 * nm, sc = (int64_t)B * sb;
  for (int b0 = 0; b0 < B; b0 += 16) {
    const int nb = min(16, B - b0);
    __syncthreads();
    // four modes per thread (nm is a multiple of 4); K entries beyond the channels are zero
    for (int i = tid; i < 32 * KC * nb * 2 * (kMixModes / 4); i += NTH) {
      const int mq = i % (kMixModes / 4), row = i / (kMixModes / 4), q = row & 1, bb = (row >> 1) % nb, ci = (row >> 1) / nb;
      const int64_t mode = m0 + 4 * mq;
      const f4 x = mode < nm && ci < W ? *reinterpret_cast<const f4*>(in + ci * sc + (b0 + bb) * sb + q * nm + mode) : zero4();
#pragma unroll
      for (int u = 0; u < 4; ++u) sI[((q * kMixModes + 4 * mq + u) * 16 + bb) * LD + ci] = bits(x[u]);
    }
    __syncthreads();
    f4 re_[2][NT], im_[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int mode = 2 * w + i;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        f4 rr = zero4(), ii = zero4(), ri = zero4(), ir = zero4();
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
          const bf8 re = lds8(sI + (mode * 16 + c) * LD + 32 * kc + 8 * g);
          const bf8 im = lds8(sI + ((kMixModes + mode) * 16 + c) * LD + 32 * kc + 8 * g);
          rr = mfma(re, r[i][0][nt][kc], rr);
          ii = mfma(im, r[i][1][nt][kc], ii);
          ri = mfma(re, r[i][1][nt][kc], ri);
          ir = mfma(im, r[i][0][nt][kc], ir);
        }
        re_[i][nt] = rr + s_re * ii;
        im_[i][nt] = ir + s_im * ri;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float* o = sO + ((16 * nt + c) * 16 + 4 * g + v) * LO + 2 * w + i;
          o[0] = re_[i][nt][v];
          o[16 * NT * 16 * LO] = im_[i][nt][v];
        }
    __syncthreads();
    for (int i = tid; i < W * nb * 2 * (kMixModes / 4); i += NTH) {
      const int mq = i % (kMixModes / 4), row = i / (kMixModes / 4), q = row & 1, bb = (row >> 1) % nb, co = (row >> 1) / nb;
      const int64_t mode = m0 + 4 * mq;
      const float* o = sO + ((q * 16 * NT + co) * 16 + bb) * LO + 4 * mq;
      if (mode < nm) *reinterpret_cast<f4*>(out + co * sc + (b0 + bb) * sb + q * nm + mode) = f4{o[0], o[1], o[2], o[3]};
    }
  }
}

// dR_re = sum_b in_re dY_re + in_im dY_im, dR_im = sum_b in_re dY_im - in_im dY_re
// per mode (in as the rows, dY as the columns), 16 batch entries per step of a
// 16x16x16 product; work split as in k_mix. Bound by the write of dR and the
// reads of in and dY.
typedef short s4 __attribute__((ext_vector_type(4)));

template <int NT>
__global__ __launch_bounds__(64 * kMixWaves) void k_mix_grad(int B, int W, int64_t nm, const float* in,
                                                             const float* dY, float* dR) {
  constexpr int LD = 16 + 4, NTH = 64 * kMixWaves, ROWS = 16 * NT;
  extern __shared__ __align__(16) unsigned char smem[];
  u16* sI = reinterpret_cast<u16*>(smem);  // [in, dY][re, im][mode][channel][b]
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int64_t m0 = (int64_t)blockIdx.x * kMixModes;
  f4 rr[2][NT][NT], ri[2][NT][NT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
      for (int y = 0; y < NT; ++y) rr[i][x][y] = ri[i][x][y] = zero4();
  for (int i = tid; i < 4 * kMixModes * ROWS * LD; i += NTH) sI[i] = 0;
  const int64_t sb = 2 * nm, sc = (int64_t)B * sb;
  for (int b0 = 0; b0 < B; b0 += 16) {
    __syncthreads();
    for (int i = tid; i < 2 * W * 16 * 2 * (kMixModes / 4); i += NTH) {
      const int mq = i % (kMixModes / 4), row = i / (kMixModes / 4), q = row & 1, bb = (row >> 1) & 15;
      const int cw = row >> 5, which = cw >= W, ch = which ? cw - W : cw;
      const int64_t mode = m0 + 4 * mq;
      const f4 x = mode < nm && b0 + bb < B
                       ? *reinterpret_cast<const f4*>((which ? dY : in) + ch * sc + (b0 + bb) * sb + q * nm + mode)
                       : zero4();
#pragma unroll
      for (int u = 0; u < 4; ++u) sI[(((2 * which + q) * kMixModes + 4 * mq + u) * ROWS + ch) * LD + bb] = bits(x[u]);
    }
    __syncthreads();
    auto frag = [&](int which, int q, int mode, int tile) {
      return *reinterpret_cast<const s4*>(sI + (((2 * which + q) * kMixModes + mode) * ROWS + 16 * tile + c) * LD + 4 * g);
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int mode = 2 * w + i;
#pragma unroll
      for (int x = 0; x < NT; ++x) {
        const s4 ar = frag(0, 0, mode, x), ai = frag(0, 1, mode, x);
        const s4 an = ai ^ (short)0x8000;  // -in_im
#pragma unroll
        for (int y = 0; y < NT; ++y) {
          const s4 br = frag(1, 0, mode, y), bi = frag(1, 1, mode, y);
          rr[i][x][y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, br, rr[i][x][y], 0, 0, 0);
          rr[i][x][y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ai, bi, rr[i][x][y], 0, 0, 0);
          ri[i][x][y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, bi, ri[i][x][y], 0, 0, 0);
          ri[i][x][y] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(an, br, ri[i][x][y], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t mode = m0 + 2 * w + i;
    if (mode >= nm) continue;
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
      for (int y = 0; y < NT; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int ci = 16 * x + 4 * g + v, co = 16 * y + c;
          if (ci >= W || co >= W) continue;
          dR[(mode * W + ci) * W + co] = rr[i][x][y][v];
          dR[((nm + mode) * W + ci) * W + co] = ri[i][x][y][v];
        }
  }
}

// ---------------------------------------------------------------------------
// A layer's output from the mixed spectrum after the inverse along x, and its
// input: for 16 rows y of one (b, x) and all channels
//   V[o][y][(p, kt)] = sum_k G_p[y][k] V2[o][k][kt],
//   s[o][y][t] = sum V[o][y][(p, kt)] Bt((p, kt), t),
//   z = s + Wm v (+ bias), a = gelu(z) or z.
// For 16 channels at a time the wavefronts first share out the channels and
// leave s in LDS, then they share out the points, where the channel product is
// formed from the fragments of v that each keeps in registers, and s added. The
// activations are read and written once (the chain of products moved z five
// times); bound by these.
struct YtArgs {
  int64_t B, X;
  int Y, T, m, W;
  const float* V2;              // [W][B][X][4m][m]
  const float *G0, *G1, *Bt;    // G_p(y, k), Bt(k, t)
  int64_t sGm, sGk, sBk, sBn;
  const float *Wm, *v;          // Wm(o, i), v [W][B][X][Y][T]
  int64_t sWo, sWi;
  const float* bias;            // may be null
  float *z, *a;                 // each may be null; a: act(z)
  int act;
};

// bytes of LDS before s[o][point]: Wm and the wavefronts' V
__host__ __device__ constexpr int yt_head(int MT) { return 2 * (16 * MT * (32 * ((MT + 1) / 2) + 8) + 4 * 16 * 40); }

template <int MT, int NTL, bool V4>
__global__ __launch_bounds__(256) void k_idft_yt(YtArgs q) {
  constexpr int KC = (MT + 1) / 2, LW = 32 * KC + 8, LV = 32 + 8;
  constexpr bool LATE = NTL * KC <= 2;  // the loads of v stay in flight over the first transforms
  extern __shared__ __align__(16) unsigned char smem[];
  const int T = q.T, m = q.m, W = q.W, Y = q.Y, NTt = (T + 15) / 16;
  const int lp = 16 * T + 4;                                     // points per channel in LDS, padded
  u16* sW = reinterpret_cast<u16*>(smem);                        // Wm[o][i]
  u16* sV = sW + 16 * MT * LW + (threadIdx.x >> 6) * 16 * LV;    // this wavefront's V[y][(p, kt)]
  float* sS = reinterpret_cast<float*>(smem + yt_head(MT));      // s[o][point] of 16 channels
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int ytiles = (Y + 15) / 16;
  const int64_t bx = blockIdx.x / ytiles;
  const int y0 = int(blockIdx.x - bx * ytiles) * 16, ny = min(16, Y - y0);
  const int64_t BX = q.B * q.X, S = BX * Y * T, pbase = (bx * Y + y0) * T;
  const int np = ny * T;
  // this wavefront's points 64 (w + 4 i) + 4c.. of all input channels
  f4 x[NTL][KC][8];
  bf8 b[NTL][KC][4];
#pragma unroll
  for (int i = 0; i < NTL; ++i)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ci = 32 * kc + 8 * g + j;
        x[i][kc][j] = ci < W ? load4<V4>(q.v + (int64_t)ci * S + pbase, 64 * (w + 4 * i) + 4 * c, np) : zero4();
      }
  auto convert = [&]() {
#pragma unroll
    for (int i = 0; i < NTL; ++i)
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const f4(&r)[8] = x[i][kc];
          b[i][kc][u] = pack8(f8{r[0][u], r[1][u], r[2][u], r[3][u], r[4][u], r[5][u], r[6][u], r[7][u]});
        }
  };
  if constexpr (!LATE) convert();
  stage(sW, q.Wm, q.sWo, q.sWi, W, W, 16 * MT, 32 * KC, LW, tid, 256);
  for (int i = lane; i < 16 * LV; i += 64) sV[i] = 0;
  // transform fragments: G_p rows y0.., K = 4m in up to two steps; Bt columns t
  const int GC = (4 * m + 31) / 32;
  bf8 ag[2][2], bt[NTL];
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    f8 x0, x1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 32 * kc + 8 * g + j;
      const bool ok = k < 4 * m && c < ny;
      x0[j] = ok ? q.G0[(y0 + c) * q.sGm + k * q.sGk] : 0.0f;
      x1[j] = ok ? q.G1[(y0 + c) * q.sGm + k * q.sGk] : 0.0f;
    }
    ag[0][kc] = pack8(x0);
    ag[1][kc] = pack8(x1);
  }
#pragma unroll
  for (int nt = 0; nt < NTL; ++nt) {
    f8 y;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 8 * g + j, t = 16 * nt + c;
      y[j] = (k < 2 * m && t < T) ? q.Bt[k * q.sBk + t * q.sBn] : 0.0f;
    }
    bt[nt] = pack8(y);
  }
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    // transforms of channels 16 mt + 4 w .. + 3, their spectra requested together
    f8 sp[4][2];
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        const int o = 16 * mt + 4 * w + h;
        const float* V2 = q.V2 + ((int64_t)o * BX + bx) * 4 * m * m;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 32 * kc + 8 * g + j;
          sp[h][kc][j] = (o < W && k < 4 * m && c < m) ? V2[k * m + c] : 0.0f;
        }
      }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      if (16 * mt + 4 * w + h >= W) continue;
      f4 a0 = zero4(), a1 = zero4();
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        if (kc >= GC) continue;
        const bf8 f = pack8(sp[h][kc]);
        a0 = mfma(ag[0][kc], f, a0);
        a1 = mfma(ag[1][kc], f, a1);
      }
      if (c < m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sV[(4 * g + r) * LV + c] = bits(a0[r]);
          sV[(4 * g + r) * LV + m + c] = bits(a1[r]);
        }
      }
      wave_sync();
      const bf8 av = lds8(sV + c * LV + 8 * g);
      float* s = sS + (4 * w + h) * lp;
#pragma unroll
      for (int nt = 0; nt < NTL; ++nt) {
        if (nt >= NTt) continue;
        const f4 acc = mfma(av, bt[nt], zero4());
        const int t = 16 * nt + c;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t < T) s[(4 * g + r) * T + t] = acc[r];
      }
      wave_sync();
    }
    if (LATE && mt == 0) convert();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NTL; ++i) {
      const int p = 64 * (w + 4 * i) + 4 * c;
      f4 acc[4] = {zero4(), zero4(), zero4(), zero4()};
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        const bf8 a = lds8(sW + (16 * mt + c) * LW + 32 * kc + 8 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = mfma(a, b[i][kc][u], acc[u]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = 16 * mt + 4 * g + r;
        if (o >= W || p >= np) continue;
        const f4 s = *reinterpret_cast<const f4*>(sS + (4 * g + r) * lp + p);
        f4 z;
#pragma unroll
        for (int u = 0; u < 4; ++u) z[u] = s[u] + acc[u][r];
        if (q.bias) z += q.bias[o];
        const int64_t off = (int64_t)o * S + pbase;
        if (q.z) store4<V4>(q.z + off, p, np, z);
        if (q.a) {
          if (q.act) z = f4{gelu(z[0]), gelu(z[1]), gelu(z[2]), gelu(z[3])};
          store4<V4>(q.a + off, p, np, z);
        }
      }
    }
    __syncthreads();
  }
}

int yt_lds(int W, int T) { return yt_head((W + 15) / 16) + 4 * 16 * (16 * T + 4); }
int head_bwd_lds(int KC, int HC) {
  const int LD = 128 * HC + 8, LP = 72;
  return 2 * (64 * LD + 128 * HC * LP + 32 * KC * LP + 32 * KC * LD);
}
int mix_lds(int NT) {
  return std::max(2 * 2 * kMixModes * 16 * (32 * ((NT + 1) / 2) + 8), 4 * 2 * 16 * NT * 16 * (kMixModes + 1));
}
int mix_grad_lds(int NT) { return 2 * 4 * kMixModes * 16 * NT * 20; }
int x_lds(int M, int K, int mats, int parts) { return 2 * (mats * up(M, 16) + parts * kXCols) * (up(K, 32) + 8); }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
template <class... P>
bool vec4(int64_t n, const P*... p) { return n % 4 == 0 && (... && aligned16(p)); }

constexpr int kCus = 256;
unsigned blocks(int64_t tasks, int per_cu) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(tasks, (int64_t)kCus * per_cu));
}

int done() { return hipGetLastError() == hipSuccess ? 0 : -3; }

// launch with lds bytes of dynamic LDS
template <auto K, class... A>
int launch(unsigned grid, int threads, int lds, void* stream, A... args) {
  if (lds > 64 * 1024 && seis::raise_lds_limit<K>(kLds) != hipSuccess) return -3;
  hipLaunchKernelGGL(K, dim3(grid), dim3(threads), lds, (hipStream_t)stream, args...);
  return done();
}

// zeroes of up to three arrays
__global__ void k_clear(int n0, float* x0, int n1, float* x1, int n2, float* x2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n0) x0[i] = 0.0f;
  if (i < n1) x1[i] = 0.0f;
  if (i < n2) x2[i] = 0.0f;
}
int clear(int64_t n0, float* x0, int64_t n1, float* x1, int64_t n2, float* x2, void* stream) {
  const int64_t n = std::max(n0, std::max(n1, n2));
  hipLaunchKernelGGL(k_clear, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, (int)n0, x0, (int)n1,
                     x1, (int)n2, x2);
  return done();
}

}  // namespace

extern "C" {

int fno_fused_shape(int64_t X, int64_t Y, int64_t T, int64_t cin, int64_t W, int64_t m, int64_t H) {
  if (X < 1 || Y < 1 || T < 1 || cin < 1 || W < 1 || m < 1 || H < 1) return 0;
  if (X > kMaxXY || Y > kMaxXY || T > kMaxT || cin > kMaxW || W > kMaxW || m > kMaxModes || H > kMaxH) return 0;
  if (2 * TyLds((int)Y, (int)T, (int)m).total > kLds || yt_lds((int)W, (int)T) > kLds) return 0;
  if (x_lds((int)(4 * m), (int)X, 2, 2) > kLds || x_lds((int)X, (int)(4 * m), 2, 1) > kLds) return 0;
  return 1;
}

int fno_pointwise(int64_t n, int64_t cout, int64_t cin, const float* Wm, const float* x, const float* bias, float* z,
                  void* stream) {
  if (n < 0 || cout < 1 || cin < 1 || cout > kMaxW || cin > kMaxW || !Wm || !x || !bias || !z) return -1;
  if (n == 0) return 0;
  const unsigned grid = blocks((n + 255) / 256, 8);
  const bool v = vec4(n, x, z);
  switch ((cout + 15) / 16) {
#define FNO_PW(MT)                                                                                               \
  case MT:                                                                                                       \
    return v ? launch<k_pointwise<MT, true>>(grid, 256, 0, stream, n, (int)cout, (int)cin, Wm, x, bias, z)       \
             : launch<k_pointwise<MT, false>>(grid, 256, 0, stream, n, (int)cout, (int)cin, Wm, x, bias, z);
    FNO_PW(1) FNO_PW(2) FNO_PW(3)
#undef FNO_PW
  }
  return -1;
}

int fno_head(int64_t n, int64_t W, int64_t H, const float* Q1, const float* q1, const float* Q2, const float* q2,
             const float* v, float* y, void* stream) {
  if (n < 0 || W < 1 || H < 1 || W > kMaxW || H > kMaxH || !Q1 || !q1 || !Q2 || !q2 || !v || !y) return -1;
  if (n == 0) return 0;
  const unsigned grid = blocks((n + 63) / 64, 4);
  const bool a = vec4(n, v);
#define FNO_HEAD(KC, HC)                                                                                            \
  if ((W + 31) / 32 == KC && (H + 127) / 128 == HC)                                                                 \
    return a ? launch<k_head<KC, HC, true>>(grid, 256, 2 * 2 * 64 * (128 * HC + 8), stream, n, (int)W, (int)H, Q1, q1, Q2, q2, v, y)          \
             : launch<k_head<KC, HC, false>>(grid, 256, 2 * 2 * 64 * (128 * HC + 8), stream, n, (int)W, (int)H, Q1, q1, Q2, q2, v, y);
  FNO_HEAD(1, 1) FNO_HEAD(1, 2) FNO_HEAD(2, 1) FNO_HEAD(2, 2)
#undef FNO_HEAD
  return -1;
}

int fno_head_backward(int64_t n, int64_t W, int64_t H, const float* Q1, const float* q1, const float* Q2,
                      const float* v, const float* dy, float* dv, float* dQ1, float* dq1, float* dQ2, void* stream) {
  if (n < 0 || W < 1 || H < 1 || W > kMaxW || H > kMaxH || !Q1 || !q1 || !Q2 || !v || !dy || !dv || !dQ1 || !dq1 || !dQ2)
    return -1;
  const int rc = clear(W * H, dQ1, H, dq1, H, dQ2, stream);
  if (rc || n == 0) return rc;
  // at least eight tiles per work-group, so that the sums it adds to memory do not outweigh its work
  const unsigned grid = blocks((n + 511) / 512, 2);
  const bool a = vec4(n, v, dy);
#define FNO_HEADB(KC, HC)                                                                                              \
  if ((W + 31) / 32 == KC && (H + 127) / 128 == HC)                                                                    \
    return a ? launch<k_head_bwd<KC, HC, true>>(grid, 256, head_bwd_lds(KC, HC), stream, n, (int)W, (int)H, Q1, q1,    \
                      Q2, v, dy, dv, dQ1, dq1, dQ2)                                                                    \
             : launch<k_head_bwd<KC, HC, false>>(grid, 256, head_bwd_lds(KC, HC), stream, n, (int)W, (int)H, Q1, q1,   \
                      Q2, v, dy, dv, dQ1, dq1, dQ2);
  FNO_HEADB(1, 1) FNO_HEADB(1, 2) FNO_HEADB(2, 1) FNO_HEADB(2, 2)
#undef FNO_HEADB
  return -1;
}

int fno_layer_backward(int64_t n, int64_t cout, int64_t cin, const float* z, const float* da, const float* x,
                       float* dz, float* dW, float* db, void* stream) {
  if (n < 0 || cout < 1 || cin < 1 || cout > kMaxW || cin > kMaxW || !da || !x || !dW || !db || (z && !dz)) return -1;
  const int rc = clear(cout * cin, dW, cout, db, 0, nullptr, stream);
  if (rc || n == 0) return rc;
  // at least four tiles per wavefront, as in fno_head_backward
  const unsigned grid = blocks((n + 1023) / 1024, 2);
  const bool v = vec4(n, da, x) && (!z || vec4(n, z, dz));
  const int MT = int(cout + 15) / 16, NT = int(cin + 15) / 16;
#define FNO_LB(M_, N_)                                                                                                \
  if (MT == M_ && NT <= N_) {                                                                                         \
    const int co = (int)cout, ci = (int)cin;                                                                          \
    if (z)                                                                                                            \
      return v ? launch<k_layer_bwd<M_, N_, true, true>>(grid, 256, 0, stream, n, co, ci, z, da, x, dz, dW, db)       \
               : launch<k_layer_bwd<M_, N_, true, false>>(grid, 256, 0, stream, n, co, ci, z, da, x, dz, dW, db);     \
    return v ? launch<k_layer_bwd<M_, N_, false, true>>(grid, 256, 0, stream, n, co, ci, z, da, x, dz, dW, db)        \
             : launch<k_layer_bwd<M_, N_, false, false>>(grid, 256, 0, stream, n, co, ci, z, da, x, dz, dW, db);      \
  }
  FNO_LB(1, 1) FNO_LB(2, 1) FNO_LB(3, 1) FNO_LB(2, 2) FNO_LB(3, 3) FNO_LB(1, 3) FNO_LB(2, 3)
#undef FNO_LB
  return -1;
}

int fno_dft_ty(int64_t slices, int64_t Y, int64_t T, int64_t m, const float* v, const float* Bt, int64_t sBk,
               int64_t sBn, const float* F0, const float* F1, int64_t sFm, int64_t sFk, float* out, void* stream) {
  if (slices < 0 || Y < 1 || T < 1 || m < 1 || Y > kMaxXY || T > kMaxT || m > kMaxModes || !v || !Bt || !F0 || !F1 || !out)
    return -1;
  if (slices == 0) return 0;
  const TyArgs a{slices, (int)Y, (int)T, (int)m, v, Bt, F0, F1, sBk, sBn, sFm, sFk, out};
  const int lds = 2 * TyLds(a.Y, a.T, a.m).total;
  if (lds > kLds) return -1;
  const unsigned grid = blocks((slices + 3) / 4, 8);
  const bool v4 = vec4(T, v);
  if (T <= 32) return v4 ? launch<k_dft_ty<1, true>>(grid, 256, lds, stream, a) : launch<k_dft_ty<1, false>>(grid, 256, lds, stream, a);
  return v4 ? launch<k_dft_ty<2, true>>(grid, 256, lds, stream, a) : launch<k_dft_ty<2, false>>(grid, 256, lds, stream, a);
}

int fno_dft_x(int64_t batch, int64_t M, int64_t K, int64_t inner, int inverse, const float* A0, const float* A1,
              int64_t sAm, int64_t sAk, const float* in, float* out, void* stream) {
  if (batch < 0 || M < 1 || K < 1 || inner < 2 || inner % 2 || !A0 || !A1 || !in || !out) return -1;
  if (M > kMaxXY || K > kMaxXY || (reinterpret_cast<uintptr_t>(in) & 7)) return -1;
  if (batch == 0) return 0;
  const int parts = inverse ? 1 : 2, nq = inverse ? 2 : 1;
  const int lds = x_lds((int)M, (int)K, 2, parts);
  if (lds > kLds) return -1;
  XArgs a{batch, (int)M, (int)K, (int)inner, parts, nq, A0, A1, sAm, sAk, in, out, M * inner * nq, inner, inner * nq};
  return launch<k_dft_x>(blocks(batch * ((inner + kXCols - 1) / kXCols), 8), 256, lds, stream, a);
}

int fno_mix(int64_t B, int64_t W, int64_t nm, const float* in, const float* R, int64_t sRi, int64_t sRo, int conj,
            float* out, void* stream) {
  if (B < 0 || W < 1 || W > kMaxW || nm < 4 || nm % 4 || B > (1 << 20) || !in || !R || !out) return -1;
  if (!aligned16(in) || !aligned16(out)) return -1;
  if (B == 0) return 0;
  const unsigned grid = (unsigned)((nm + kMixModes - 1) / kMixModes);
  const float s = conj ? 1.0f : -1.0f;
  switch ((W + 15) / 16) {
#define FNO_MIX(NT) \
  case NT: return launch<k_mix<NT>>(grid, 64 * kMixWaves, mix_lds(NT), stream, (int)B, (int)W, nm, in, R, sRi, sRo, s, -s, out);
    FNO_MIX(1) FNO_MIX(2) FNO_MIX(3)
#undef FNO_MIX
  }
  return -1;
}

int fno_mix_grad(int64_t B, int64_t W, int64_t nm, const float* in, const float* dY, float* dR, void* stream) {
  if (B < 0 || W < 1 || W > kMaxW || nm < 4 || nm % 4 || B > (1 << 20) || !in || !dY || !dR) return -1;
  if (!aligned16(in) || !aligned16(dY)) return -1;
  const unsigned grid = (unsigned)((nm + kMixModes - 1) / kMixModes);
  switch ((W + 15) / 16) {
#define FNO_MG(NT) \
  case NT: return launch<k_mix_grad<NT>>(grid, 64 * kMixWaves, mix_grad_lds(NT), stream, (int)B, (int)W, nm, in, dY, dR);
    FNO_MG(1) FNO_MG(2) FNO_MG(3)
#undef FNO_MG
  }
  return -1;
}

int fno_idft_yt(int64_t B, int64_t X, int64_t Y, int64_t T, int64_t m, int64_t W, const float* V2, const float* G0,
                const float* G1, int64_t sGm, int64_t sGk, const float* Bt, int64_t sBk, int64_t sBn, const float* Wm,
                int64_t sWo, int64_t sWi, const float* v, const float* bias, float* z, float* a, int act,
                void* stream) {
  if (B < 0 || X < 1 || Y < 1 || T < 1 || m < 1 || W < 1 || X > kMaxXY || Y > kMaxXY || T > kMaxT || m > kMaxModes ||
      W > kMaxW || !V2 || !G0 || !G1 || !Bt || !Wm || !v || (!z && !a))
    return -1;
  const int64_t grid = B * X * ((Y + 15) / 16);
  const int lds = yt_lds((int)W, (int)T);
  if (lds > kLds || grid > (int64_t(1) << 31) - 1) return -1;
  if (B == 0) return 0;
  const YtArgs q{B, X, (int)Y, (int)T, (int)m, (int)W, V2, G0, G1, Bt, sGm, sGk, sBk, sBn, Wm, v, sWo, sWi, bias, z, a, act};
  // rows of 16 T points, so every tile starts aligned where a (b, x) plane does
  const bool v4 = vec4(Y * T, v) && (!z || aligned16(z)) && (!a || aligned16(a));
#define FNO_YT(MT, NTL)                                                                         \
  if ((W + 15) / 16 == MT && (T + 15) / 16 <= NTL)                                              \
    return v4 ? launch<k_idft_yt<MT, NTL, true>>((unsigned)grid, 256, lds, stream, q)           \
              : launch<k_idft_yt<MT, NTL, false>>((unsigned)grid, 256, lds, stream, q);
  FNO_YT(1, 1) FNO_YT(2, 1) FNO_YT(3, 1) FNO_YT(1, 2) FNO_YT(2, 2) FNO_YT(3, 2) FNO_YT(1, 4) FNO_YT(2, 4) FNO_YT(3, 4)
#undef FNO_YT
  return -1;
}

}  // extern "C"
