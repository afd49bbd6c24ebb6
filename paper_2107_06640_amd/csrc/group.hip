// Group kernels (group.hpp): one work-group per 16 elements.
//
// LDS holds the 16 elements' rows as [row][quantity][element]. A contraction
// with a reference matrix is a chain of 16x16x4 products whose columns are the
// 16 elements, one product per quantity; A fragments come from global memory
// in fragment order (one coalesced load each, cached), B fragments are rows of
// LDS, and a wavefront holds the results of the quantities it needs side by
// side, so that the per-element work that mixes quantities is lane-local:
//   * the star matrices follow the contraction (they act on quantities, K^d on
//     rows): the stress rows of (K^d)^T D need the three velocity products of
//     each d, the velocity rows the six stress products, so a task is one row
//     tile of either kind and reads each row of LDS once for all three d;
//   * a face trace task holds all nine quantities of 16 nodes: hand-over and
//     Godunov flux follow in registers.
// Result register v of lane group g is row 16t + 4v + g in both precisions:
// the FP64 product orders its rows so, and the FP32 product's A rows are
// permuted to it.
#include "group.hpp"

#include <algorithm>

#include "elastic.hpp"
#include "layout.hpp"
#include "lds_limit.hpp"

namespace seis {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Vec;
template <>
struct Vec<float> {
  using type = f4;
};
template <>
struct Vec<double> {
  using type = d4;
};
template <typename T>
using V4 = typename Vec<T>::type;

__device__ __forceinline__ f4 mma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ d4 mma(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Sizes of degree N: slabs of four K entries, 16-row tiles, rows of LDS.
template <int N>
struct Dim {
  static constexpr int B = nbasis(N), Bf = nface(N), B1 = nbasis(N - 1);
  static constexpr int RT = row_tiles(B), RT1 = row_tiles(B1), FT = row_tiles(Bf);
  static constexpr int SB = (B + 3) / 4, S1 = (B1 + 3) / 4, NS = (Bf + 3) / 4;
  // fragment image: K^d transposed [d][slab][tile], K^d [d][slab][tile], E_f [f][slab][tile], L_f [f][slab][tile]
  static constexpr int oK = 0, oV = oK + 3 * SB * RT1, oE = oV + 3 * S1 * RT, oL = oE + 4 * SB * FT;
  static constexpr int frags = oL + 4 * NS * RT;
  static constexpr int rows(int k) { return nbasis(N - k); }  // rows of the k-th derivative
  static constexpr int row0(int k) {                          // its first row in LDS
    int r = 0;
    for (int j = 0; j < k; ++j) r += nbasis(N - j);
    return r;
  }
  static constexpr int drows = row0(N + 1), wrows = 4 * 4 * NS;
  static constexpr int lds_rows = drows > wrows ? drows : wrows;  // (the last level, one row, is no slab's source)
};

constexpr int kRow = 9 * 16;  // values of one row of 16 elements

// Wavefronts of a work-group: two tasks per row tile at the upper orders, fewer
// where there are fewer tiles; FP64 at order 5 has room for two work-groups of
// four wavefronts per CU.
template <typename T, int N>
constexpr int waves = N >= 5 || (N == 4 && sizeof(T) == 4) ? 8 : 4;

// A fragments of the first slabs of a contraction, requested before the barrier
// that its rows wait for.
constexpr int kAhead = 3;

template <typename T, int ND>
struct First {
  T a[kAhead][ND];
  __device__ __forceinline__ void load(const T* img, int sd, int ss, int S) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
#pragma unroll
      for (int d = 0; d < ND; ++d) a[s][d] = img[d * sd + (s < S ? s : 0) * ss];
  }
};

// acc[d][r] += sum over S slabs of A_d (fragments img + d sd + slab ss, the first
// kAhead slabs in f) times rows of NR quantities of src (its element and lane group
// included), quantity r at Q[r]; rows from nin on count as zero. A fragments are
// requested kAhead slabs ahead (two slabs measured 11% slower on the whole order-6
// predictor: a slab of few products is shorter than the latency of L2), rows one slab
// ahead; one scheduling region per slab keeps the requests there.
template <typename T, int ND, int NR, int S, int nin>
__device__ __forceinline__ void contract(V4<T> (&acc)[ND][NR], const First<T, ND>& f, const T* img, int sd, int ss,
                                         const T* src, const int (&Q)[NR], int g) {
  T a[kAhead + 1][ND], x[2][NR];
#pragma unroll
  for (int s = 0; s < kAhead && s < S; ++s)
#pragma unroll
    for (int d = 0; d < ND; ++d) a[s][d] = f.a[s][d];
#pragma unroll
  for (int r = 0; r < NR; ++r) x[0][r] = src[Q[r] * 16];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if (s + kAhead < S) {
#pragma unroll
      for (int d = 0; d < ND; ++d) a[(s + kAhead) % (kAhead + 1)][d] = img[d * sd + (s + kAhead) * ss];
    }
    if (s + 1 < S) {
#pragma unroll
      for (int r = 0; r < NR; ++r) x[(s + 1) & 1][r] = src[(s + 1) * 4 * kRow + Q[r] * 16];
    }
    T(&xs)[NR] = x[s & 1];
    if (nin % 4 && s == S - 1) {
#pragma unroll
      for (int r = 0; r < NR; ++r) xs[r] = 4 * s + g < nin ? xs[r] : T(0);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int d = 0; d < ND; ++d) acc[d][r] = mma(a[s % (kAhead + 1)][d], xs[r], acc[d][r]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename T, int ND, int NR>
__device__ __forceinline__ void clear(V4<T> (&acc)[ND][NR]) {
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[d][r] = V4<T>{T(0), T(0), T(0), T(0)};
}

// Kind of a task: the products its rows read and the rows it writes. A
// velocity task reads stresses, a stress task velocities.
template <bool VEL>
struct Kind {
  static constexpr int NR = VEL ? 6 : 3, NP = VEL ? 3 : 6, P0 = VEL ? 6 : 0, R0 = VEL ? 0 : 6;
};
template <int NR>
struct Seq {
  int v[NR];
  constexpr Seq(int q0) : v() {
    for (int i = 0; i < NR; ++i) v[i] = q0 + i;
  }
};

// sum_e A_e w_e with w_e = sum_d G[d][e] y_d at register v: the three velocity
// components from the stress products, or the stress components from the three
// velocity products.
template <typename T, bool VEL>
__device__ __forceinline__ void star_of(const V4<T> (&y)[3][Kind<VEL>::NR], int v, const T (&G)[9], T lam, T mu, T rinv,
                                        T (&out)[Kind<VEL>::NP]) {
  auto w = [&](int e, int r) { return G[e] * y[0][r][v] + G[3 + e] * y[1][r][v] + G[6 + e] * y[2][r][v]; };
  if constexpr (VEL) {
    out[0] = -rinv * (w(0, 0) + w(1, 3) + w(2, 5));
    out[1] = -rinv * (w(0, 3) + w(1, 1) + w(2, 4));
    out[2] = -rinv * (w(0, 5) + w(1, 4) + w(2, 2));
  } else {
    const T xx = w(0, 0), yy = w(1, 1), zz = w(2, 2), tr = lam * (xx + yy + zz), m2 = T(2) * mu;
    out[0] = -(tr + m2 * xx);
    out[1] = -(tr + m2 * yy);
    out[2] = -(tr + m2 * zz);
    out[3] = -mu * (w(0, 1) + w(1, 0));
    out[4] = -mu * (w(1, 2) + w(2, 1));
    out[5] = -mu * (w(0, 2) + w(2, 0));
  }
}

// Task of a wavefront at level K: velocity tasks (the longer ones)
// first; the levels with few tasks start from other
// wavefronts, so that no SIMD gets the long task of every level.
template <typename T, int N, int K>
__device__ __forceinline__ int ck_task(int w) {
  constexpr int TO = row_tiles(Dim<N>::rows(K + 1));
  if (K == 0 || TO > 2 || w > 3) return w;
  return TO == 2 ? (w + 2) & 3 : 3 - w;
}

// Cauchy-Kowalevski levels K..N-1: rows of derivative K + 1 from those of
// derivative K; f holds the first A fragments of this wavefront's task. From
// level 1 on, the wavefronts without a task add the source derivative to the
// time integral, I~ += D_K / (K + 1) in place of D0, which no product reads any
// more (each level in its own barrier interval, so no two add to a row at once).
template <typename T, int N, int K>
__device__ __forceinline__ void ck_levels(T* lds, const T* img, First<T, 3>& f, int w, int lane, const T (&G)[9], T lam,
                                          T mu, T rinv) {
  using D = Dim<N>;
  constexpr int NW = waves<T, N>, sd = D::SB * D::RT1 * 64, ss = D::RT1 * 64;
  if constexpr (K < N) {
    constexpr int nin = D::rows(K), nout = D::rows(K + 1), S = (nin + 3) / 4, TO = row_tiles(nout);
    const int el = lane & 15, g = lane >> 4;
    const T* src = lds + D::row0(K) * kRow;
    T* dst = lds + D::row0(K + 1) * kRow;
    const T fk = T(-1) / T(K + 1);
    auto task = [&](auto kind, int t) {
      using Kd = Kind<decltype(kind)::value>;
      V4<T> y[3][Kd::NR];
      clear<T>(y);
      constexpr Seq<Kd::NR> q(Kd::R0);
      contract<T, 3, Kd::NR, S, nin>(y, f, img + (D::oK + t) * 64 + lane, sd, ss, src + g * kRow + el, q.v, g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * t + 4 * v + g;
        T out[Kd::NP];
        star_of<T, decltype(kind)::value>(y, v, G, lam, mu, rinv, out);
        if (row < nout)
#pragma unroll
          for (int p = 0; p < Kd::NP; ++p) dst[row * kRow + (Kd::P0 + p) * 16 + el] = fk * out[p];
      }
    };
    const int i0 = ck_task<T, N, K>(w);
    if (i0 < TO) task(std::true_type{}, i0);
    else if (i0 < 2 * TO) task(std::false_type{}, i0 - TO);
    if constexpr (2 * TO > NW) {  // a second round (at most one more task each)
      static_assert(2 * TO <= 2 * NW, "more tasks than two rounds");
      const int i = i0 + NW;
      if (i < 2 * TO) {
        f.load(img + (D::oK + (i < TO ? i : i - TO)) * 64 + lane, sd, ss, S);
        if (i < TO) task(std::true_type{}, i);
        else task(std::false_type{}, i - TO);
      }
    }
    if constexpr (K >= 1) {
      constexpr int busy = 2 * TO, idle = NW - busy;
      static_assert(idle > 0, "a level with a task for every wavefront has nobody to add its source");
      if (i0 >= busy) {
        const T wk = T(1) / T(K + 1);
        for (int i = (i0 - busy) * 64 + lane; i < nin * kRow; i += idle * 64) lds[i] += wk * src[i];
      }
    }
    if constexpr (K + 1 < N) {
      constexpr int TN = row_tiles(D::rows(K + 2)), SN = (nout + 3) / 4;
      const int i = ck_task<T, N, K + 1>(w);
      f.load(img + (D::oK + (i < TN ? i : (i < 2 * TN ? i - TN : 0))) * 64 + lane, sd, ss, SN);
    }
    __syncthreads();
    ck_levels<T, N, K + 1>(lds, img, f, w, lane, G, lam, mu, rinv);
  }
}

// Predictor: Cauchy-Kowalevski levels, time integral, volume term, face traces
// with hand-over and own-trace flux, lifts (Sec. 4.1 and 4.2). Bound by the chain
// of levels, each behind a barrier (45% of the cycles at order 6), and by the requests of A
// fragments from L2. FP64, 23 562 elements at order 5 with LTS: 0.63 ms a
// macro step, 2.7 in the plain form (corrector: 0.19 and 0.9). Persistent
// work-groups that request the next rows of Q during the lift took 0.67.
template <typename T, int N>
__global__ __launch_bounds__((64 * waves<T, N>), sizeof(T) == 8 ? 2 : (N <= 5 ? 4 : 2)) void k_predict_group(
    GroupArgs<T> a, int64_t e0, int64_t e1, Sched sc) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t grp = (e0 >> 4) + xcd_block();
  using D = Dim<N>;
  constexpr int B = D::B, Bf = D::Bf, RT = D::RT, FT = D::FT, NW = waves<T, N>, NT = 64 * NW;
  constexpr int LN = (D::SB * 9 + NW - 1) / NW;
  const int tid = threadIdx.x, lane = tid & 63, el = lane & 15, g = lane >> 4;
  const int64_t e = grp * 16 + el;
  const bool live = e >= e0 && e < e1;
  const int64_t ec = live ? e : e0;
  T* Qg = a.Q + grp * (int64_t)(RT * 36 * 64);
  // line i = (slab, quantity) of the tiled rows of Q, four rows: all of a wavefront's lines
  // are requested before the first is stored
  T ql[LN];
#pragma unroll
  for (int j = 0; j < LN; ++j) ql[j] = w + j * NW < D::SB * 9 ? Qg[(w + j * NW) * 64 + lane] : T(0);
  T G[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) G[i] = a.G[ec * 9 + i];
  const T lam = a.mat[ec * 3], mu = a.mat[ec * 3 + 1], rinv = a.mat[ec * 3 + 2];
  const int ds = live ? a.dslot[ec] : -1;
  const int hs = __builtin_amdgcn_readfirstlane(a.hslot[grp]);
  First<T, 3> f3;
  {
    constexpr int TO = row_tiles(D::rows(1));
    const int i = ck_task<T, N, 0>(w);
    f3.load(a.img + (D::oK + (i < TO ? i : (i < 2 * TO ? i - TO : 0))) * 64 + lane, D::SB * D::RT1 * 64, D::RT1 * 64, D::SB);
  }
#pragma unroll
  for (int j = 0; j < LN; ++j) {
    const int i = w + j * NW, row = 4 * (i / 9) + g;
    if (i < D::SB * 9 && row < B) lds[row * kRow + (i % 9) * 16 + el] = ql[j];
  }
  __syncthreads();
  const bool anyd = __any(ds >= 0);
  if (anyd && ds >= 0) {  // D0 of elements with a gravity or fault face, before I~ takes its place
    T* gd = a.gD + (int64_t)ds * (N + 1) * B * 9;
    for (int i = tid; i < B * kRow; i += NT) {
      const int row = i / kRow, q = (i / 16) % 9;
      gd[row * 9 + q] = lds[i];
    }
  }
  if (hs >= 0) {  // the same for groups with a finer neighbour: the half-step integral starts from D0
    T* h = a.Ih + (int64_t)hs * (RT * 36 * 64);
    for (int i = tid; i < B * kRow; i += NT) {
      const int row = i / kRow, q = (i / 16) % 9;
      h[((row >> 2) * 9 + q) * 64 + el + 16 * (row & 3)] = lds[i];
    }
  }
  if (anyd || hs >= 0) __syncthreads();
  ck_levels<T, N, 0>(lds, a.img, f3, w, lane, G, lam, mu, rinv);
  // the last derivative (one row) completes I~
  constexpr int oN = D::row0(N) * kRow;
  if (tid < kRow) lds[tid] += (T(1) / T(N + 1)) * lds[oN + tid];
  if (anyd && ds >= 0) {
    T* gd = a.gD + (int64_t)ds * (N + 1) * B * 9;
#pragma unroll
    for (int k = 1; k <= N; ++k)
      for (int i = tid; i < D::rows(k) * kRow; i += NT) {
        const int row = i / kRow, q = (i / 16) % 9;
        gd[k * B * 9 + row * 9 + q] = lds[D::row0(k) * kRow + i];
      }
  }
  if (hs >= 0) {
    // the first half of the step: D0 + sum_k Dk 2^-k/(k+1)
    T* h = a.Ih + (int64_t)hs * (RT * 36 * 64);
    for (int i = tid; i < B * kRow; i += NT) {
      const int row = i / kRow, q = (i / 16) % 9;
      T* hp = h + ((row >> 2) * 9 + q) * 64 + el + 16 * (row & 3);
      T y = *hp, pw = T(1);
#pragma unroll
      for (int k = 1; k <= N; ++k) {
        pw *= T(0.5);
        if (row < D::rows(k)) y += lds[D::row0(k) * kRow + i] * (pw * (T(1) / T(k + 1)));
      }
      *hp = y;
    }
  }
  // volume: each wavefront keeps the increment of its (tile, kind) tasks
  constexpr int TPW = (2 * RT + NW - 1) / NW;
  constexpr int vsd = D::S1 * RT * 64, vss = RT * 64;
  f3.load(a.img + (D::oV + (w < RT ? w : (w < 2 * RT ? w - RT : 0))) * 64 + lane, vsd, vss, D::S1);
  __syncthreads();
  V4<T> dq[TPW][6];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    const int i = w + u * NW;
#pragma unroll
    for (int p = 0; p < 6; ++p) dq[u][p] = V4<T>{T(0), T(0), T(0), T(0)};
    if (u > 0 && i < 2 * RT) f3.load(a.img + (D::oV + (i < RT ? i : i - RT)) * 64 + lane, vsd, vss, D::S1);
    auto task = [&](auto kind, int t) {
      using Kd = Kind<decltype(kind)::value>;
      V4<T> y[3][Kd::NR];
      clear<T>(y);
      constexpr Seq<Kd::NR> q(Kd::R0);
      contract<T, 3, Kd::NR, D::S1, 4 * D::S1>(y, f3, a.img + (D::oV + t) * 64 + lane, vsd, vss, lds + g * kRow + el, q.v, g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        T out[Kd::NP];
        star_of<T, decltype(kind)::value>(y, v, G, lam, mu, rinv, out);
#pragma unroll
        for (int p = 0; p < Kd::NP; ++p) dq[u][p][v] = out[p];
      }
    };
    if (i < RT) task(std::true_type{}, i);
    else if (i < 2 * RT) task(std::false_type{}, i - RT);
  }
  // traces at the nodes of (face, node tile) tasks, from the last wavefront down
  constexpr int TPT = (4 * FT + NW - 1) / NW;
  T fl[TPT][4][9];
  const int mh = a.mh4[ec], parity = sc.parity(ec);
#pragma unroll
  for (int u = 0; u < TPT; ++u) {
    const int j = (NW - 1 - w) + u * NW;
    if (j >= 4 * FT) continue;
    const int f = j / FT, nt = j - f * FT;
    First<T, 1> f1;
    f1.load(a.img + (D::oE + f * D::SB * FT + nt) * 64 + lane, 0, FT * 64, D::SB);
    T c[11];
#pragma unroll
    for (int i = 0; i < 11; ++i) c[i] = a.RCm[(ec * 4 + f) * 12 + i];
    const int32_t tgt = a.tgt[ec * 4 + f];
    V4<T> va[1][9];
    clear<T>(va);
    constexpr Seq<9> q(0);
    contract<T, 1, 9, D::SB, 4 * D::SB>(va, f1, a.img + (D::oE + f * D::SB * FT + nt) * 64 + lane, 0, FT * 64,
                                        lds + g * kRow + el, q.v, g);
    const int md = (mh >> (8 * f)) & 3, h = (mh >> (8 * f + 2)) & 7;
    const bool send = live && md != 0, half = md == MODE_COARSER;
    const int32_t tg = send ? tgt : 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int node = 16 * nt + 4 * v + g;
      if (16 * nt + 4 * v >= Bf) {  // no node of the register exists
#pragma unroll
        for (int p = 0; p < 9; ++p) fl[u][v][p] = T(0);
        continue;
      }
      T t9[9];
#pragma unroll
      for (int p = 0; p < 9; ++p) t9[p] = va[0][p][v];
      if (send && node < Bf) {
        // the neighbour's node numbering and time step: a coarser one gets the halves of this element's
        // two steps added up, a finer one the full-step trace that launch_finer splits
        const int mr = a.pinv[h * Bf + node];
        T* blk = a.In + in_block(tg >> 2, tg & 3, mr, FT) * 576;
        const int l = in_lane(tg >> 2, mr);
        const T s = half ? T(0.5) : T(1);
        V4<T>* d8 = reinterpret_cast<V4<T>*>(blk + 8 * l);
        V4<T> lo = {s * t9[0], s * t9[1], s * t9[2], s * t9[3]}, hi = {s * t9[4], s * t9[5], s * t9[6], s * t9[7]};
        T last = s * t9[8];
        if (half && parity) {  // one writer per slot
          lo += d8[0];
          hi += d8[1];
          last += blk[512 + l];
        }
        d8[0] = lo;
        d8[1] = hi;
        blk[512 + l] = last;
      }
      T out[9];
      node_flux(c, lam, mu, rinv, t9, out);
#pragma unroll
      for (int p = 0; p < 9; ++p) fl[u][v][p] = node < Bf ? out[p] : T(0);
    }
  }
  constexpr int NR4 = 4 * D::NS;  // rows per face
  __syncthreads();  // every trace has read I~: the fluxes take its place
#pragma unroll
  for (int u = 0; u < TPT; ++u) {
    const int j = (NW - 1 - w) + u * NW;
    if (j >= 4 * FT) continue;
    const int f = j / FT, nt = j - f * FT;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (16 * nt + 4 * v >= NR4) continue;
      const int node = 16 * nt + 4 * v + g;
#pragma unroll
      for (int p = 0; p < 9; ++p) lds[(f * NR4 + node) * kRow + p * 16 + el] = fl[u][v][p];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    const int i = w + u * NW;
    auto lift = [&](auto kind, int t) {
      using Kd = Kind<decltype(kind)::value>;
      V4<T> acc[1][Kd::NP];
#pragma unroll
      for (int p = 0; p < Kd::NP; ++p) acc[0][p] = dq[u][p];
      constexpr Seq<Kd::NP> s(Kd::P0);
      First<T, 1> f1;
      f1.load(a.img + (D::oL + t) * 64 + lane, 0, RT * 64, 4 * D::NS);
      T q[4][Kd::NP];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int p = 0; p < Kd::NP; ++p)
          q[v][p] = 16 * t + 4 * v < B ? Qg[((t * 4 + v) * 9 + Kd::P0 + p) * 64 + lane] : T(0);
      // the faces follow one another in the image and in LDS
      contract<T, 1, Kd::NP, 4 * D::NS, 16 * D::NS>(acc, f1, a.img + (D::oL + t) * 64 + lane, 0, RT * 64,
                                                    lds + g * kRow + el, s.v, g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (!live || 16 * t + 4 * v + g >= B) continue;
        T* o = Qg + (t * 4 + v) * 9 * 64 + lane;
#pragma unroll
        for (int p = 0; p < Kd::NP; ++p) o[(Kd::P0 + p) * 64] = q[v][p] + acc[0][p][v];
      }
    };
    if (i < RT) lift(std::true_type{}, i);
    else if (i < 2 * RT) lift(std::false_type{}, i - RT);
  }
}

// Corrector: Q -= sum_f L_f flux(neighbour trace of face f); on the second step
// of a pair a face towards a coarser neighbour reads its second-half trace.
template <typename T, int N>
__global__ __launch_bounds__((64 * waves<T, N>), sizeof(T) == 8 ? 2 : 4) void k_correct_group(GroupArgs<T> a, int64_t e0,
                                                                                         int64_t e1, Sched sc) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t grp = (e0 >> 4) + xcd_block();
  using D = Dim<N>;
  constexpr int B = D::B, Bf = D::Bf, RT = D::RT, FT = D::FT, NW = waves<T, N>, NR4 = 4 * D::NS;
  const int lane = threadIdx.x & 63, el = lane & 15, g = lane >> 4;
  const int64_t e = grp * 16 + el;
  const bool live = e >= e0 && e < e1;
  const int64_t ec = live ? e : e0;
  const T lam = a.mat[ec * 3], mu = a.mat[ec * 3 + 1], rinv = a.mat[ec * 3 + 2];
  const int parity = sc.parity(ec);
  T* Qg = a.Q + grp * (int64_t)(RT * 36 * 64);
  for (int j = w; j < 4 * FT; j += NW) {
    const int f = j / FT, nt = j - f * FT;
    const int h2 = parity ? a.rhalf2[ec * 4 + f] : -1;
    T in[4][9];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int node = 16 * nt + 4 * v + g;
      if (16 * nt + 4 * v >= Bf) continue;
      const T* blk = a.In + ((grp * 4 + f) * FT * 4 + nt * 4 + v) * 576;
      if (h2 >= 0 && node < Bf) {
        const T* s = a.H2 + ((int64_t)h2 * Bf + node) * 9;
#pragma unroll
        for (int p = 0; p < 9; ++p) in[v][p] = s[p];
      } else {
        const V4<T>* d8 = reinterpret_cast<const V4<T>*>(blk + 8 * lane);
        const V4<T> lo = d8[0], hi = d8[1];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          in[v][p] = lo[p];
          in[v][4 + p] = hi[p];
        }
        in[v][8] = blk[512 + lane];
      }
    }
    T c[11];
#pragma unroll
    for (int i = 0; i < 11; ++i) c[i] = a.RCp[(ec * 4 + f) * 12 + i];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int node = 16 * nt + 4 * v + g;
      if (16 * nt + 4 * v >= NR4) continue;
      T out[9];
      node_flux(c, lam, mu, rinv, in[v], out);
#pragma unroll
      for (int p = 0; p < 9; ++p)
        lds[(f * NR4 + node) * kRow + p * 16 + el] = node < Bf ? out[p] : T(0);
    }
  }
  // tasks: a row tile and the first five or the last four quantities
  for (int i = w; i < 2 * RT; i += NW) {
    const int t = i < RT ? i : i - RT;
    auto lift = [&](auto first, bool sync) {
      constexpr int I0 = decltype(first)::value ? 0 : 5, NP = decltype(first)::value ? 5 : 4;
      First<T, 1> f1;
      f1.load(a.img + (D::oL + t) * 64 + lane, 0, RT * 64, 4 * D::NS);
      T q[4][NP];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int p = 0; p < NP; ++p)
          q[v][p] = 16 * t + 4 * v < B ? Qg[((t * 4 + v) * 9 + (I0 + p)) * 64 + lane] : T(0);
      if (sync) __syncthreads();
      V4<T> dq[1][NP];
      clear<T>(dq);
      constexpr Seq<NP> s(I0);
      contract<T, 1, NP, 4 * D::NS, 16 * D::NS>(dq, f1, a.img + (D::oL + t) * 64 + lane, 0, RT * 64, lds + g * kRow + el, s.v, g);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (!live || 16 * t + 4 * v + g >= B) continue;
        T* o = Qg + (t * 4 + v) * 9 * 64 + lane;
#pragma unroll
        for (int p = 0; p < NP; ++p) o[(I0 + p) * 64] = q[v][p] + dq[0][p][v];
      }
    };
    // every wavefront passes the barrier with its first task, or below if it has none
    if (i < RT) lift(std::true_type{}, i == w);
    else lift(std::false_type{}, i == w);
  }
  if (w >= 2 * RT) __syncthreads();
}

// Half-step traces of a group's faces towards finer neighbours: the predictor
// wrote the full-step trace V into the neighbour's inbox; h1 = E_f I~_h (I~_h
// the integral over the first half, of the whole group in LDS) replaces it and
// 2 V - h1, the second half, goes to the neighbour's slot. A thread takes two
// nodes of a face, so that each value of I~_h read from LDS is used twice; the
// node-contiguous matrices (Et) keep the nodes of a face on distinct banks. V is
// requested before the products, which hide the chain face -> target -> inbox.
// Every h1 is one sum over the modes in ascending order.
constexpr int kFinerThreads = 256;

template <typename T, int N>
__global__ __launch_bounds__(kFinerThreads) void k_finer_group(GroupArgs<T> a, int64_t first) {
  using D = Dim<N>;
  constexpr int B = D::B, Bf = D::Bf, RT = D::RT, FT = D::FT, PAIRS = (Bf + 1) / 2;
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char smem[];
  T* sI = reinterpret_cast<T*>(smem);  // tiled layout of the group
  T* sE = sI + D::SB * 9 * 64;         // [f][mode][node]
  const int32_t* ent = a.fix_group + (first + xcd_block()) * 3;
  const int grp = ent[0], f0 = ent[1], nf = ent[2];
  auto stage = [&](T* dst, const T* src, int n) {
    for (int i = threadIdx.x; i < n * (int)sizeof(T) / 16; i += kFinerThreads)
      reinterpret_cast<u4*>(dst)[i] = reinterpret_cast<const u4*>(src)[i];
  };
  stage(sE, a.Et, 4 * B * Bf);
  stage(sI, a.Ih + (int64_t)a.hslot[grp] * (RT * 36 * 64), D::SB * 9 * 64);
  __syncthreads();
  for (int i = threadIdx.x; i < nf * PAIRS; i += kFinerThreads) {
    const int id = a.fix_list[f0 + i / PAIRS], m0 = i % PAIRS, m1 = m0 + PAIRS < Bf ? m0 + PAIRS : m0;
    const int64_t e = id >> 2;
    const int f = id & 3;
    const int32_t tg = a.tgt[id], slot = a.half2[id];
    const int hp = (a.mh4[e] >> (8 * f + 2)) & 7;
    T *blk[2], *out[2];
    int l8[2];
    T V[2][9], h[2][9];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int mr = a.pinv[hp * Bf + (u ? m1 : m0)];
      blk[u] = a.In + in_block(tg >> 2, tg & 3, mr, FT) * 576;
      l8[u] = in_lane(tg >> 2, mr);
      out[u] = a.H2 + ((int64_t)slot * Bf + mr) * 9;
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        V[u][p] = p < 8 ? blk[u][8 * l8[u] + p] : blk[u][512 + l8[u]];
        h[u][p] = T(0);
      }
    }
    const T *E0 = sE + f * B * Bf, *I = sI + (int)(e & 15);
#pragma unroll 4
    for (int l = 0; l < B; ++l) {
      const T x0 = E0[l * Bf + m0], x1 = E0[l * Bf + m1];
      const T* Il = I + (l >> 2) * 576 + 16 * (l & 3);
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        const T y = Il[p * 64];
        h[0][p] += x0 * y;
        h[1][p] += x1 * y;
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (u == 1 && m1 == m0) continue;
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        blk[u][p < 8 ? 8 * l8[u] + p : 512 + l8[u]] = h[u][p];
        out[u][p] = T(2) * V[u][p] - h[u][p];
      }
    }
  }
}

template <auto K, class... A>
hipError_t launch(unsigned grid, int threads, int lds, hipStream_t s, A... args) {
  if (lds > 64 * 1024) {
    const hipError_t st = raise_lds_limit<K>(160 * 1024);
    if (st != hipSuccess) return st;
  }
  hipLaunchKernelGGL(K, dim3(grid), dim3(threads), lds, s, args...);
  return hipGetLastError();
}

unsigned groups_of(int64_t e0, int64_t e1) { return (unsigned)(((e1 - 1) >> 4) - (e0 >> 4) + 1); }

template <typename T, int N>
hipError_t pred(const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc, hipStream_t s) {
  using D = Dim<N>;
  constexpr int lds = D::lds_rows * kRow * (int)sizeof(T);
  static_assert(lds <= 160 * 1024, "the group's rows exceed the LDS of a CU");
  return launch<k_predict_group<T, N>>(groups_of(e0, e1), 64 * waves<T, N>, lds, s, a, e0, e1, sc);
}
template <typename T, int N>
hipError_t corr(const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc, hipStream_t s) {
  using D = Dim<N>;
  constexpr int lds = D::wrows * kRow * (int)sizeof(T);
  return launch<k_correct_group<T, N>>(groups_of(e0, e1), 64 * waves<T, N>, lds, s, a, e0, e1, sc);
}
template <typename T, int N>
hipError_t finer(const GroupArgs<T>& a, int64_t first, int64_t n, hipStream_t s) {
  using D = Dim<N>;
  constexpr int lds = (D::SB * 9 * 64 + 4 * D::Bf * D::B) * (int)sizeof(T);
  static_assert(lds <= 160 * 1024, "the half-step images exceed the LDS of a CU");
  return launch<k_finer_group<T, N>>((unsigned)n, kFinerThreads, lds, s, a, first);
}

template <int N>
std::vector<double> image(const Model& M, bool fp64) {
  using D = Dim<N>;
  std::vector<double> r((size_t)D::frags * 64, 0.0);
  // lane l of a fragment: A row l % 16 (permuted for FP32, see above), K entry l / 16
  auto fill = [&](int frag, int tile, int slab, int rows, int ks, auto at) {
    for (int l = 0; l < 64; ++l) {
      const int c = l & 15, i = 16 * tile + (fp64 ? c : tile_perm(c)), k = 4 * slab + (l >> 4);
      if (i < rows && k < ks) r[(size_t)frag * 64 + l] = at(i, k);
    }
  };
  const auto& R = M.ref;
  for (int d = 0; d < 3; ++d) {
    for (int s = 0; s < D::SB; ++s)
      for (int t = 0; t < D::RT1; ++t)
        fill(D::oK + (d * D::SB + s) * D::RT1 + t, t, s, D::B1, D::B,
             [&](int m, int l) { return R.K[((size_t)d * D::B + l) * D::B + m]; });
    for (int s = 0; s < D::S1; ++s)
      for (int t = 0; t < D::RT; ++t)
        fill(D::oV + (d * D::S1 + s) * D::RT + t, t, s, D::B, D::B1,
             [&](int k, int l) { return R.K[((size_t)d * D::B + k) * D::B + l]; });
  }
  for (int f = 0; f < 4; ++f) {
    for (int s = 0; s < D::SB; ++s)
      for (int t = 0; t < D::FT; ++t)
        fill(D::oE + (f * D::SB + s) * D::FT + t, t, s, D::Bf, D::B,
             [&](int m, int l) { return R.E[((size_t)f * D::Bf + m) * D::B + l]; });
    for (int s = 0; s < D::NS; ++s)
      for (int t = 0; t < D::RT; ++t)
        fill(D::oL + (f * D::NS + s) * D::RT + t, t, s, D::B, D::Bf,
             [&](int k, int m) { return R.L[((size_t)f * D::B + k) * D::Bf + m]; });
  }
  return r;
}

}  // namespace

std::vector<double> group_image(const Model& M, bool fp64) {
  switch (M.N) {
    case 2: return image<2>(M, fp64);
    case 3: return image<3>(M, fp64);
    case 4: return image<4>(M, fp64);
    case 5: return image<5>(M, fp64);
    case 6: return image<6>(M, fp64);
  }
  return {};
}

#define SEIS_GROUP(FN, ...)                                      \
  switch (N) {                                                   \
    case 2: return FN<T, 2>(__VA_ARGS__);                        \
    case 3: return FN<T, 3>(__VA_ARGS__);                        \
    case 4: return FN<T, 4>(__VA_ARGS__);                        \
    case 5: return FN<T, 5>(__VA_ARGS__);                        \
    case 6:                                                      \
      if constexpr (group_order<T>(6)) return FN<T, 6>(__VA_ARGS__); \
  }                                                              \
  return hipErrorInvalidValue;

template <typename T>
hipError_t launch_predict_group(int N, const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc,
                                hipStream_t s) {
  if (e1 <= e0) return hipSuccess;
  SEIS_GROUP(pred, a, e0, e1, sc, s)
}
template <typename T>
hipError_t launch_correct_group(int N, const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc,
                                hipStream_t s) {
  if (e1 <= e0) return hipSuccess;
  SEIS_GROUP(corr, a, e0, e1, sc, s)
}
template <typename T>
hipError_t launch_finer(int N, const GroupArgs<T>& a, int64_t first, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  SEIS_GROUP(finer, a, first, n, s)
}

template hipError_t launch_predict_group<float>(int, const GroupArgs<float>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_predict_group<double>(int, const GroupArgs<double>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_correct_group<float>(int, const GroupArgs<float>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_correct_group<double>(int, const GroupArgs<double>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_finer<float>(int, const GroupArgs<float>&, int64_t, int64_t, hipStream_t);
template hipError_t launch_finer<double>(int, const GroupArgs<double>&, int64_t, int64_t, hipStream_t);

}  // namespace seis
