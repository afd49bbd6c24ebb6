// Plain element kernels: one work-group per element, every contraction a
// loop over shared memory and reference matrices read from global memory.
// They are the straightforward form of the update (the baseline the tuned
// kernels are measured against) and serve FP64 and FP32.
//
// Predictor (Sec. 4.1, Taylor expansion and Cauchy-Kowalevski procedure),
// with scaled derivatives Dk = dt^k/k! d^kQ/dt^k:
//   D0 = Q,  D(k+1) = -1/(k+1) sum_d (K^d)^T Dk (dt A*_d)^T
//   I~ = I/dt = sum_k Dk/(k+1)
// Element-local corrector part (Sec. 4.1 semi-discrete form; Sec. 4.2 flux):
//   Q += sum_d K^d I~ (dt A*_d)^T - sum_i L_i (F~-_i (E_i I~))
// where E_i evaluates traces at the face nodes and L_i lifts nodal values.
// Neighbour part (corrector): Q -= sum_i L_i (F~+_i In_i).
#include "device.hpp"
#include "elastic.hpp"
#include "layout.hpp"

namespace seis {

namespace {

// Threads per element: 128 for throughput, as many as the longest loops have
// items, so that more work-groups share a CU (a pass of BF16 steps at order 6 whose finest cluster of
// 1971 elements runs here took 8.76 ms; 192 and 256 threads 9.05, 512 10.0); a launch
// over a few elements (a tiny LTS cluster) is bound by the latency of one
// work-group, so it uses 1024, or 256 at the lowest orders (threads_for).
// The thread count is a launch parameter of one compiled kernel, not a
// template argument, so that an element's arithmetic (and its rounding) is
// the same whichever launch covers it.
constexpr int NT_WIDE = 128, NT_TALL = 1024, TALL_BELOW = 256;

// LDS rows of nine quantities are three padded triples, each one wide read. A
// contraction item is a (row, triple) whose sums run side by side; GROUP items
// that read the same LDS rows (the directions of K, faces, two row halves) share
// a thread where there are elements enough to fill the chip, so that a read of
// LDS feeds 3 GROUP products: what bounds these loops is the return path of
// LDS and of the matrices' loads, not the products. A launch over a few elements keeps
// one item per thread, and so do the orders whose longest loop has no more items
// than the work-group threads (kOneItem): there sharing only lengthens the
// chains. A step in FP32 of 600 / 29 478 elements, shared and one item per thread: order 3
// 17.5 / 186 us and 15.0 / 167, order 4 23.0 / 303 and 20.4 / 268, order 5 34.6 / 507 and
// 32.2 / 524. Matrices are indexed with the row contiguous, one coalesced
// load. Every sum runs in ascending order on its own, however the
// items are shared out.
constexpr int kPad = 12;
template <int N>
constexpr bool kOneItem = 9 * nbasis(N - 1) <= NT_WIDE;  // orders 2..4
__device__ __forceinline__ int padded(int row, int p) { return row * kPad + p / 3 * 4 + p % 3; }

template <typename T>
struct alignas(4 * sizeof(T)) Triple {
  T v[4];
};

// Modes requested together: eight (four: 1.5% on that pass); twelve where that measured faster, in
// the one-item form of orders 5 and 6, which only launches over few elements take (LTS box of 576
// elements, a launch per cluster, a macro step in FP32: order 5 365 us with eight, 335 with twelve;
// order 6 474 and 427; order 7 562 and 606), and at order 2, whose longest sum that is (152 and 142).
template <int GROUP, int N>
constexpr int kAhead = GROUP == 1 && (N == 1 || N == 4 || N == 5) ? 12 : 8;

// acc[u][j] += sum_l m[u][l ld] row_l[j], l < n, of the triple at x
template <int GROUP, int N, typename T>
__device__ __forceinline__ void chain(T (&acc)[GROUP][3], const T* const (&m)[GROUP], int ld, const T* x, int n) {
  constexpr int U = kAhead<GROUP, N>;
#pragma unroll U
  for (int l = 0; l < n; ++l) {
    const Triple<T> r = *reinterpret_cast<const Triple<T>*>(x + l * kPad);
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      const T k = m[u][l * ld];
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[u][j] += k * r.v[j];
    }
  }
}
// the same, subtracted
template <int GROUP, int N, typename T>
__device__ __forceinline__ void chain_sub(T (&acc)[GROUP][3], const T* const (&m)[GROUP], int ld, const T* x, int n) {
  constexpr int U = kAhead<GROUP, N>;
#pragma unroll U
  for (int l = 0; l < n; ++l) {
    const Triple<T> r = *reinterpret_cast<const Triple<T>*>(x + l * kPad);
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      const T k = m[u][l * ld];
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[u][j] -= k * r.v[j];
    }
  }
}

// Y_d = (K^d)^T D (rows below nout), GROUP directions per thread
template <int GROUP, typename T, int N>
__device__ __forceinline__ void plain_level(const DevData<T>& d, const T* sD, T* sY, int nin, int nout) {
  constexpr int B = nbasis(N), B1 = nbasis(N - 1);
  for (int i = threadIdx.x; i < 9 / GROUP * nout; i += blockDim.x) {
    const int gp = i / nout, m = i - gp * nout, d0 = gp / 3 * GROUP, pg = gp % 3;
    T acc[GROUP][3] = {};
    const T* K[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) K[u] = d.K + (size_t)(d0 + u) * B * B + m;
    chain<GROUP, N>(acc, K, B, sD + pg * 4, nin);
#pragma unroll
    for (int u = 0; u < GROUP; ++u)
#pragma unroll
      for (int j = 0; j < 3; ++j) sY[((d0 + u) * B1 + m) * kPad + pg * 4 + j] = acc[u][j];
  }
}

// traces of the first sets of (s0, s1) at the face nodes, GROUP faces per thread
template <int GROUP, typename T, int N>
__device__ __forceinline__ void plain_trace(const DevData<T>& d, int sets, const T* s0, T* sV0, const T* s1, T* sV1) {
  constexpr int B = nbasis(N), Bf = nface(N), NI = 12 / GROUP * Bf;
  for (int j = threadIdx.x; j < sets * NI; j += blockDim.x) {
    const int i = j < NI ? j : j - NI, gp = i / Bf, m = i % Bf, f0 = gp / 3 * GROUP, pg = gp % 3;
    const T* s = j < NI ? s0 : s1;
    T* sV = j < NI ? sV0 : sV1;
    T acc[GROUP][3] = {};
    const T* E[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) E[u] = d.Et + (size_t)(f0 + u) * B * Bf + m;
    chain<GROUP, N>(acc, E, Bf, s + pg * 4, B);
#pragma unroll
    for (int u = 0; u < GROUP; ++u)
#pragma unroll
      for (int j = 0; j < 3; ++j) sV[((f0 + u) * Bf + m) * kPad + pg * 4 + j] = acc[u][j];
  }
}

// Q += volume term of sY (if VOLUME), then minus the lifts of the fluxes sF; GROUP rows per thread.
template <int GROUP, bool VOLUME, typename T, int N>
__device__ __forceinline__ void plain_lift(const DevData<T>& d, int64_t e, const T* sY, const T* sF) {
  constexpr int B = nbasis(N), B1 = nbasis(N - 1), Bf = nface(N), RT = row_tiles(B), H = (B + GROUP - 1) / GROUP;
  for (int i = threadIdx.x; i < 3 * H; i += blockDim.x) {
    const int pg = i / H, k0 = i % H;
    int row[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) row[u] = k0 + u * H < B ? k0 + u * H : B - 1;
    T acc[GROUP][3] = {};
    const T* M[GROUP];
    if constexpr (VOLUME) {
      for (int dd = 0; dd < 3; ++dd) {
#pragma unroll
        for (int u = 0; u < GROUP; ++u) M[u] = d.Kt + (size_t)dd * B * B + row[u];
        chain<GROUP, N>(acc, M, B, sY + dd * B1 * kPad + pg * 4, B1);
      }
    }
    // the faces follow one another
#pragma unroll
    for (int u = 0; u < GROUP; ++u) M[u] = d.Lt + row[u];
    if constexpr (VOLUME)
      chain_sub<GROUP, N>(acc, M, B, sF + pg * 4, 4 * Bf);
    else
      chain<GROUP, N>(acc, M, B, sF + pg * 4, 4 * Bf);
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      if (k0 + u * H >= B) continue;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        T& q = d.Q[qidx(e, row[u], pg * 3 + j, RT)];
        if constexpr (VOLUME)
          q += acc[u][j];
        else
          q -= acc[u][j];
      }
    }
  }
}

// Predictor of one element. 1971 elements at order 6 in FP32: 122 us with one
// product per read of LDS and of the matrices, 103 us in this form, 91 us
// with the elements of a group on one XCD (corrector: 35, 33 and 26 us).
template <typename T, int N>
__global__ __launch_bounds__(NT_TALL) void k_predict_plain(DevData<T> d, int64_t e0, Sched sc) {
  const int NT = blockDim.x;
  const bool single = kOneItem<N> || NT == NT_TALL;
  constexpr int B = nbasis(N), Bf = nface(N);
  constexpr int B1 = nbasis(N - 1);
  constexpr int RT = row_tiles(B), FT = row_tiles(Bf);
  static_assert(4 * Bf >= B, "the derivative takes the traces' place");
  const int64_t e = e0 + xcd_block();
  const int parity = sc.parity(e);
  const int tid = threadIdx.x;
  __shared__ alignas(32) T sV[4 * Bf * kPad], sVh[4 * Bf * kPad];
  __shared__ alignas(32) T sI[B * kPad], sIh[B * kPad];
  __shared__ alignas(32) T sY[3 * B1 * kPad];  // reused for the volume term
  __shared__ T sG[9], sM[3];
  T* sD = sV;  // until the traces
  if (tid < 9) sG[tid] = d.G[e * 9 + tid];
  if (tid < 3) sM[tid] = d.mat[e * 3 + tid];
  const int gs = d.dslot[e];
  T* gD = gs >= 0 ? d.gD + (int64_t)gs * (N + 1) * B * 9 : nullptr;
  // the half-step integral, for a face towards a finer neighbour: one of the four modes (bytes, 0..3)
  // is 2. One load: four behind || follow one another.
  const unsigned md4 = *reinterpret_cast<const unsigned*>(d.mode + e * 4);
  const bool finer = (md4 & ~(md4 << 1) & 0x02020202u) != 0;
  for (int i = tid; i < B * 9; i += NT) {
    const T q = d.Q[qidx(e, i / 9, i % 9, RT)];
    const int x = padded(i / 9, i % 9);
    sD[x] = q;
    sI[x] = q;
    sIh[x] = q;
    if (gD) gD[i] = q;
  }
  __syncthreads();
  const T lam = sM[0], mu = sM[1], rinv = sM[2];
  T half = T(0.5);
#pragma unroll  // sizes and divisors constant: 0.6% of the BF16 pass
  for (int k = 0; k < N; ++k) {
    const int nin = nbasis(N - k), nout = nbasis(N - k - 1);
    // Y_d = (K^d)^T D_k restricted to the non-zero rows
    if (single)
      plain_level<1, T, N>(d, sD, sY, nin, nout);
    else
      plain_level<3, T, N>(d, sD, sY, nin, nout);
    __syncthreads();
    const T f = T(-1) / T(k + 1);
    for (int i = tid; i < nout * 9; i += NT) {
      const int m = i / 9, p = i % 9;
      T wx[9], wy[9], wz[9];
      for (int r = 0; r < 9; ++r) {
        const T y0 = sY[padded(0 * B1 + m, r)], y1 = sY[padded(1 * B1 + m, r)], y2 = sY[padded(2 * B1 + m, r)];
        wx[r] = sG[0] * y0 + sG[3] * y1 + sG[6] * y2;
        wy[r] = sG[1] * y0 + sG[4] * y1 + sG[7] * y2;
        wz[r] = sG[2] * y0 + sG[5] * y1 + sG[8] * y2;
      }
      const T v = f * grad_op(p, lam, mu, rinv, wx, wy, wz);
      const int x = padded(m, p);
      sD[x] = v;
      sI[x] += v / T(k + 2);
      sIh[x] += v * half / T(k + 2);
      if (gD) gD[(k + 1) * B * 9 + i] = v;  // rows below B_{N-k-1}: the others are zero
    }
    half *= T(0.5);
    __syncthreads();
  }
  // traces at the face nodes: full step and first half step
  if (single) {
    plain_trace<1, T, N>(d, finer ? 2 : 1, sI, sV, sIh, sVh);
  } else {  // one set fills the threads
    plain_trace<2, T, N>(d, 1, sI, sV, sI, sV);
    if (finer) plain_trace<2, T, N>(d, 1, sIh, sVh, sIh, sVh);
  }
  __syncthreads();
  // hand the traces to the neighbours (in their node numbering)
  for (int i = tid; i < 4 * Bf * 9; i += NT) {
    const int f = i / (Bf * 9), m = (i / 9) % Bf, p = i % 9;
    const int md = d.mode[e * 4 + f];
    if (md == 0) continue;
    const int32_t t = d.tgt[e * 4 + f];
    const int src = padded(f * Bf + d.perm[d.hperm[e * 4 + f] * Bf + m], p);
    const T v = sV[src];
    T* dst = d.In + inidx(t >> 2, t & 3, m, p, FT);
    if (md == 1) {
      *dst = v;
    } else if (md == 2) {
      const T h1 = sVh[src];  // first half-step integral over the receiver's dt
      *dst = h1;
      d.H2[((int64_t)d.half2[e * 4 + f] * Bf + m) * 9 + p] = T(2) * v - h1;
    } else {
      *dst = parity ? *dst + T(0.5) * v : T(0.5) * v;
    }
  }
  // local flux at the nodes: F~-_f V_f (into sVh)
  __syncthreads();
  for (int i = tid; i < 4 * Bf * 9; i += NT) {
    const int f = i / (Bf * 9), m = (i / 9) % Bf, p = i % 9;
    const T* F = d.Fm + ((e * 4 + f) * 81 + p * 9);
    T a = T(0);
    for (int r = 0; r < 9; ++r) a += F[r] * sV[padded(f * Bf + m, r)];
    sVh[padded(f * Bf + m, p)] = a;
  }
  // volume: Z_d[l] = (dt A*_d) I~[l] for l < B1
  for (int i = tid; i < 3 * B1; i += NT) {
    const int dd = i / B1, l = i % B1;
    T in[9], out[9];
    for (int p = 0; p < 9; ++p) in[p] = sI[padded(l, p)];
    apply_star(sG[dd * 3 + 0], sG[dd * 3 + 1], sG[dd * 3 + 2], lam, mu, rinv, in, out);
    for (int p = 0; p < 9; ++p) sY[padded(dd * B1 + l, p)] = out[p];
  }
  __syncthreads();
  if (single)
    plain_lift<1, true, T, N>(d, e, sY, sVh);
  else
    plain_lift<2, true, T, N>(d, e, sY, sVh);
}

template <typename T, int N>
__global__ __launch_bounds__(NT_TALL) void k_correct_plain(DevData<T> d, int64_t e0, Sched sc) {
  const int NT = blockDim.x;
  constexpr int Bf = nface(N);
  constexpr int FT = row_tiles(Bf);
  const int64_t e = e0 + xcd_block();
  const int parity = sc.parity(e);
  const int tid = threadIdx.x;
  __shared__ alignas(32) T sW[4 * Bf * kPad];
  for (int i = tid; i < 4 * Bf * 9; i += NT) {
    const int f = i / (Bf * 9), m = (i / 9) % Bf, p = i % 9;
    const int h2 = d.rhalf2[e * 4 + f];
    const T* F = d.Fp + ((e * 4 + f) * 81 + p * 9);
    T a = T(0);
    if (parity && h2 >= 0) {
      const T* src = d.H2 + ((int64_t)h2 * Bf + m) * 9;
      for (int r = 0; r < 9; ++r) a += F[r] * src[r];
    } else {
      for (int r = 0; r < 9; ++r) a += F[r] * d.In[inidx(e, f, m, r, FT)];
    }
    sW[padded(f * Bf + m, p)] = a;
  }
  __syncthreads();
  if (kOneItem<N> || NT == NT_TALL)
    plain_lift<1, false, T, N>(d, e, nullptr, sW);
  else
    plain_lift<2, false, T, N>(d, e, nullptr, sW);
}

// Gravity face (Sec. 4.3): per point, the forcing f = v_n + p/Z of the
// predicted solution (p = -n.s.n), the ODE d eta/dt = f - a eta, dH/dt = eta
// integrated exactly through its Taylor series over the element's step, and
// the time-integrated boundary flux (stress rows -lambda (eta1 - eta0),
// velocity rows g H n) lifted with the face rule. Bound by latency (traces,
// the series, lifts, each behind a barrier): 1152 faces at order 6 took 50 us with
// row-contiguous matrices, the zero rows of the derivatives and two FP64 divisions per
// term, 42 us in this form, 37 us with neighbouring faces on one XCD.
template <typename T, int N>
__global__ __launch_bounds__(256) void k_gravity(DevData<T> d, const int32_t* glist) {
  constexpr int B = nbasis(N);
  constexpr int RT = row_tiles(B);
  constexpr int nq = (N + 1) * (N + 1);
  const int gf = glist[xcd_block()];
  const int tid = threadIdx.x;
  const int64_t e = d.g_elem[gf];
  const int face = d.g_face[gf];
  const double* par = d.g_par + gf * 8;
  const double scale = par[0], nx = par[1], ny = par[2], nz = par[3], Z = par[4], a = par[5], lam = par[6],
               dt = par[7];
  constexpr int terms = N + 24;  // of the Taylor series
  __shared__ T sD[(N + 1) * B * 9];
  __shared__ double sFm[N + 1][nq], sF[2][nq], sStep[terms], sInv[terms];
  // the element's scaled time derivatives, staged once (coalesced): the rows of derivative k below B_{N-k}
  const T* D = d.gD + (int64_t)gf * (N + 1) * B * 9;
#pragma unroll
  for (int k = 0; k <= N; ++k)
    for (int i = tid; i < nbasis(N - k) * 9; i += 256) sD[k * B * 9 + i] = D[k * B * 9 + i];
  // the series' coefficients, once per work-group: the divisions of a point's
  // recurrence would be a chain of their own
  if (tid < terms) {
    sStep[tid] = dt / (tid + 1);
    sInv[tid] = 1.0 / (tid + 2);
  }
  __syncthreads();
  // trace of each derivative at each surface point: one (order, point) pair per
  // thread, so that a wavefront has few lengths of sum and reads the matrix coalesced
  for (int w = tid; w < nq * (N + 1); w += 256) {
    const int m = w / nq, q = w - m * nq;
    const double* Eq = d.Egt + (size_t)face * B * nq + q;
    const T* Dm = sD + m * B * 9;
    double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int rows = nbasis(N - m);
#pragma unroll 4
    for (int l = 0; l < rows; ++l) {
      const double el = Eq[l * nq];
#pragma unroll
      for (int p = 0; p < 9; ++p) v[p] += el * (double)Dm[l * 9 + p];
    }
    const double tx = v[0] * nx + v[3] * ny + v[5] * nz;
    const double ty = v[3] * nx + v[1] * ny + v[4] * nz;
    const double tz = v[5] * nx + v[4] * ny + v[2] * nz;
    const double pm = -(tx * nx + ty * ny + tz * nz);
    sFm[m][q] = v[6] * nx + v[7] * ny + v[8] * nz + pm / Z;
  }
  __syncthreads();
  for (int q = tid; q < nq; q += 256) {
    const double eta0 = d.eta[(int64_t)gf * nq + q];
    double em = eta0, eta1 = eta0, H = eta0 * dt;
    for (int m = 0; m < terms; ++m) {
      const double fm = m <= N ? sFm[m][q] : 0.0;
      em = sStep[m] * (fm - a * em);
      eta1 += em;
      // em dt / (m + 2), correctly rounded: the quotient by the reciprocal, corrected by its remainder
      // (Markstein's division)
      const double x = em * dt, r = sInv[m], y = x * r;
      H += isfinite(y) ? fma(fma(-y, double(m + 2), x), r, y) : y;
    }
    d.eta[(int64_t)gf * nq + q] = eta1;
    sF[0][q] = -lam * (eta1 - eta0);
    sF[1][q] = d.g * H;
  }
  __syncthreads();
  // lift: rows of the three normal stresses (one sum) and the velocities
  for (int i = tid; i < B * 4; i += 256) {
    const int j = i / B, kk = i - j * B;
    const double* Lq = d.Lgt + (size_t)face * nq * B + kk;
    double acc = 0.0;
    if (j == 0) {
#pragma unroll 8
      for (int q = 0; q < nq; ++q) acc += Lq[q * B] * sF[0][q];
      for (int p = 0; p < 3; ++p) d.Q[qidx(e, kk, p, RT)] -= (T)(scale * acc);
    } else {
      const double nj = j == 1 ? nx : (j == 2 ? ny : nz);
#pragma unroll 8
      for (int q = 0; q < nq; ++q) acc += Lq[q * B] * sF[1][q] * nj;
      d.Q[qidx(e, kk, 5 + j, RT)] -= (T)(scale * acc);
    }
  }
}

// Threads per element of a launch over ne elements. The one-item orders have no loop of more
// than some 300 items: 256 threads while latency bounds the launch, 128 beyond (order 3, a step in
// FP32 with 128, 256, 512 and 1024 threads: 288 elements 14.2, 13.5, 13.6, 17.5 us; 1296 elements 16.6, 16.5,
// 25, 41; 6000 elements 40, 50, 85, 151).
template <int N>
unsigned threads_for(int64_t ne) {
  if (kOneItem<N>) return ne < 1024 ? 256 : NT_WIDE;
  return ne < TALL_BELOW ? NT_TALL : NT_WIDE;
}

template <typename T, int N>
hipError_t pred_n(const DevData<T>& d, int64_t e0, int64_t ne, const Sched& sc, hipStream_t s) {
  if (ne <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_predict_plain<T, N>), dim3((unsigned)ne), dim3(threads_for<N>(ne)), 0, s, d, e0, sc);
  return hipGetLastError();
}
template <typename T, int N>
hipError_t corr_n(const DevData<T>& d, int64_t e0, int64_t ne, const Sched& sc, hipStream_t s) {
  if (ne <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_correct_plain<T, N>), dim3((unsigned)ne), dim3(threads_for<N>(ne)), 0, s, d, e0, sc);
  return hipGetLastError();
}
template <typename T, int N>
hipError_t grav_n(const DevData<T>& d, const int32_t* glist, int64_t ng, hipStream_t s) {
  if (ng <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_gravity<T, N>), dim3((unsigned)ng), dim3(256), 0, s, d, glist);
  return hipGetLastError();
}

}  // namespace

#define SEIS_DISPATCH(FN, ...)                  \
  switch (N) {                                  \
    case 1: return FN<T, 1>(__VA_ARGS__);       \
    case 2: return FN<T, 2>(__VA_ARGS__);       \
    case 3: return FN<T, 3>(__VA_ARGS__);       \
    case 4: return FN<T, 4>(__VA_ARGS__);       \
    case 5: return FN<T, 5>(__VA_ARGS__);       \
    case 6: return FN<T, 6>(__VA_ARGS__);       \
    case 7: return FN<T, 7>(__VA_ARGS__);       \
    default: return hipErrorInvalidValue;       \
  }

template <typename T>
hipError_t launch_predict_plain(int N, const DevData<T>& d, int64_t e0, int64_t ne, const Sched& sc, hipStream_t s) {
  SEIS_DISPATCH(pred_n, d, e0, ne, sc, s)
}
template <typename T>
hipError_t launch_correct_plain(int N, const DevData<T>& d, int64_t e0, int64_t ne, const Sched& sc, hipStream_t s) {
  SEIS_DISPATCH(corr_n, d, e0, ne, sc, s)
}
template <typename T>
hipError_t launch_gravity(int N, const DevData<T>& d, const int32_t* glist, int64_t ng, hipStream_t s) {
  SEIS_DISPATCH(grav_n, d, glist, ng, s)
}

template hipError_t launch_predict_plain<double>(int, const DevData<double>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_predict_plain<float>(int, const DevData<float>&, int64_t, int64_t, const Sched&,
                                                hipStream_t);
template hipError_t launch_correct_plain<double>(int, const DevData<double>&, int64_t, int64_t, const Sched&,
                                                 hipStream_t);
template hipError_t launch_correct_plain<float>(int, const DevData<float>&, int64_t, int64_t, const Sched&,
                                                hipStream_t);
template hipError_t launch_gravity<double>(int, const DevData<double>&, const int32_t*, int64_t, hipStream_t);
template hipError_t launch_gravity<float>(int, const DevData<float>&, const int32_t*, int64_t, hipStream_t);

}  // namespace seis
