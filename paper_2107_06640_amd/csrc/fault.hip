// Friction kernel of the dynamic-rupture faces (see fault.hpp).
#include "fault.hpp"

#include "elastic.hpp"
#include "layout.hpp"

namespace seis {

namespace {

// traction s n split into its normal and tangential parts, and the same for v
__device__ inline void split_state(const double* q, const double* n, double& sn, double* tt, double& vn,
                                   double* vt) {
  const double tx = q[0] * n[0] + q[3] * n[1] + q[5] * n[2];
  const double ty = q[3] * n[0] + q[1] * n[1] + q[4] * n[2];
  const double tz = q[5] * n[0] + q[4] * n[1] + q[2] * n[2];
  sn = tx * n[0] + ty * n[1] + tz * n[2];
  tt[0] = tx - sn * n[0];
  tt[1] = ty - sn * n[1];
  tt[2] = tz - sn * n[2];
  vn = q[6] * n[0] + q[7] * n[1] + q[8] * n[2];
  for (int d = 0; d < 3; ++d) vt[d] = q[6 + d] - vn * n[d];
}

// rate and state: the slip rate V in [0, T / eta] with
// T - eta V = sigma a asinh(V / (2 V0) e^(psi / a)), whose left side falls
// strictly with V; Newton steps kept inside a shrinking bracket (bisection
// where a step leaves it)
__device__ inline double rs_slip_rate(double T, double sigma, double eta, double psi, double a, double V0,
                                      double Vguess) {
  double lo = 0.0, hi = T / eta;
  const double c = exp(psi / a) / (2.0 * V0);
  double V = fmin(fmax(Vguess, lo), hi);
  for (int it = 0; it < 100; ++it) {
    const double x = c * V;
    const double g = T - eta * V - sigma * a * asinh(x);
    if (g > 0.0) lo = V; else hi = V;
    const double dg = -eta - sigma * a * c / sqrt(1.0 + x * x);
    double Vn = V - g / dg;
    if (!(Vn > lo && Vn < hi)) Vn = 0.5 * (lo + hi);
    if (fabs(Vn - V) <= 1e-15 * fmax(fabs(V), 1e-300) || hi - lo <= 1e-15 * fmax(hi, 1e-300)) {
      V = Vn;
      break;
    }
    V = Vn;
  }
  return V;
}

__device__ inline double rs_steady_state(double V, const double* r) {
  // r: a, b, L, V0, f0, f_w, V_w
  const double fLV = r[4] - (r[1] - r[0]) * log(V / r[3]);
  const double q = V / r[6], q2 = q * q, q4 = q2 * q2;
  const double fss = r[5] + (fLV - r[5]) / pow(1.0 + q4 * q4, 0.125);
  return r[0] * log(2.0 * r[3] / V * sinh(fss / r[0]));
}

// One work-group of kFaultThreads per fault face: the two elements' stored
// derivatives are staged in LDS with contiguous reads; all threads form their
// traces at the nodes, then the states of both sides at every time point,
// split along the normal, then what the law needs of them; thread m applies the law
// at node m, point after point. Bound by that serial chain of FP64 divisions and
// roots on one wavefront, so it holds nothing that does
// not depend on the point before (1152 faces at order 6, four macro steps of 55 296 elements: 2.47 ms with the
// states formed inside it and row-contiguous matrices, 2.40 in this form, 2.37 with
// registers for three wavefronts per SIMD).
constexpr int kFaultThreads = 256;

template <typename T, int N>
__global__ __launch_bounds__(kFaultThreads, 3) void k_fault(FaultArgs a, const T* gD, T* In, int64_t f0) {
  constexpr int B = nbasis(N), Bf = nface(N), FT = row_tiles(Bf);
  constexpr int ND = (N + 1) * B * 9;      // stored values per element
  constexpr int NS = 2 * (N + 1) * Bf;     // (time point, side, node)
  // derivatives D~k of the two sides, then the split states [time point][side][node][8]
  __shared__ __align__(8) unsigned char buf[2 * ND * sizeof(T) > NS * 64 ? 2 * ND * sizeof(T) : NS * 64];
  // their traces at the nodes, then (s, v_n, locked tractions) [time point][node][5]
  __shared__ double tr[2][N + 1][Bf][9];
  T(*sd)[ND] = reinterpret_cast<T(*)[ND]>(buf);
  double* split = reinterpret_cast<double*>(buf);
  const int64_t f = f0 + xcd_block();
  const int64_t em = a.elem[f], ep = a.pelem[f];
  const int fm = a.face[f], fp = a.pface[f], h = a.perm[f];
  const T* Dm = gD + (int64_t)a.dslot[em] * ND;
  const T* Dp = gD + (int64_t)a.dslot[ep] * ND;
  for (int i = threadIdx.x; i < ND; i += blockDim.x) {
    if (i % (B * 9) >= nbasis(N - i / (B * 9)) * 9) continue;  // derivative k has B_{N-k} rows, the rest is zero
    sd[0][i] = Dm[i];
    sd[1][i] = Dp[i];
  }
  __syncthreads();
  // three quantities of a node per item, the nodes of E contiguous
  for (int i = threadIdx.x; i < NS * 3; i += blockDim.x) {
    const int k = i / (6 * Bf), r = i - k * (6 * Bf), side = r / (3 * Bf), p = (r / Bf) % 3 * 3, m = r % Bf;
    const int node = side == 0 ? m : a.pinv[h * Bf + m];
    const double* Em = a.Et + (int64_t)(side == 0 ? fm : fp) * B * Bf + node;
    const T* D = &sd[side][k * B * 9 + p];
    double acc[3] = {0.0, 0.0, 0.0};
    const int rows = nbasis(N - k);
#pragma unroll 8
    for (int l = 0; l < rows; ++l) {
      const double x = Em[l * Bf];
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[j] += x * (double)D[l * 9 + j];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) tr[side][k][m][p + j] = acc[j];
  }
  __syncthreads();
  const double* g = a.geo + f * 8;
  const double n[3] = {g[0], g[1], g[2]};
  const double zpm = g[3], zsm = g[4], zpp = g[5], zsp = g[6], dt = g[7];
  const double eta = zsm * zsp / (zsm + zsp);
  for (int i = threadIdx.x; i < NS; i += blockDim.x) {
    const int j = i / (2 * Bf), side = (i / Bf) & 1, mi = i % Bf;
    const double tj = a.tq[j];
    double q[9], tt[3], vt[3], sn, vn;
    for (int p = 0; p < 9; ++p) {
      double x = 0.0, pw = 1.0;
      for (int k = 0; k <= N; ++k) {  // q(t) = sum_k D~k (t / dt)^k
        x += pw * tr[side][k][mi][p];
        pw *= tj;
      }
      q[p] = x;
    }
    split_state(q, n, sn, tt, vn, vt);
    double* o = split + i * 8;
    o[0] = sn;
    o[1] = vn;
    for (int c = 0; c < 3; ++c) {
      o[2 + c] = tt[c];
      o[5 + c] = vt[c];
    }
  }
  __syncthreads();
  double* point = &tr[0][0][0][0];
  for (int i = threadIdx.x; i < (N + 1) * Bf; i += blockDim.x) {
    const int j = i / Bf, mi = i - j * Bf;
    const double *x = split + (2 * j * Bf + mi) * 8, *y = x + Bf * 8;  // '-' and '+'
    double* o = point + i * 5;
    o[0] = (zpp * x[0] + zpm * y[0] + zpm * zpp * (y[1] - x[1])) / (zpm + zpp);
    o[1] = (zpm * x[1] + zpp * y[1] + y[0] - x[0]) / (zpm + zpp);
    for (int c = 0; c < 3; ++c) o[2 + c] = eta * (x[2 + c] / zsm + y[2 + c] / zsp + y[5 + c] - x[5 + c]);
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m >= Bf) return;
  const double* pr = a.par + f * kFaultParams;
  const double s0 = pr[0];
  const double t0n = pr[1] * n[0] + pr[2] * n[1] + pr[3] * n[2];
  const double tau0[3] = {pr[1] - t0n * n[0], pr[2] - t0n * n[1], pr[3] - t0n * n[2]};
  const double mu_s = pr[4], mu_d = pr[5], dc = pr[6], coh = pr[7];
  const bool rate_state = pr[15] == double(kLawRateState);
  double* st = a.state + (f * Bf + m) * kFaultState;
  double slip[3] = {st[0], st[1], st[2]}, psi = st[3];
  double V[3] = {st[4], st[5], st[6]}, Tb[3] = {0.0, 0.0, 0.0}, Stot = 0.0;  // V: the last slip rate
  double as = 0.0, avn = 0.0, atau[3] = {0.0, 0.0, 0.0}, avm[3] = {0.0, 0.0, 0.0}, avp[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
  for (int j = 0; j <= N; ++j) {
    const double wj = a.tw[j];
    const double *x = split + (2 * j * Bf + m) * 8, *y = x + Bf * 8, *w = point + (j * Bf + m) * 5;
    const double s = w[0], vn = w[1];
    double lock[3], Ttot[3], ttm[3], vtm[3], ttp[3], vtp[3];
    for (int d = 0; d < 3; ++d) {
      ttm[d] = x[2 + d];
      vtm[d] = x[5 + d];
      ttp[d] = y[2 + d];
      vtp[d] = y[5 + d];
      lock[d] = w[2 + d];
      Ttot[d] = tau0[d] + lock[d];
    }
    Stot = s0 + s;
    const double mag = sqrt(Ttot[0] * Ttot[0] + Ttot[1] * Ttot[1] + Ttot[2] * Ttot[2]);
    bool slips;
    double ratio;
    if (rate_state) {
      // always sliding, at the rate-dependent strength
      const double v = rs_slip_rate(mag, fmax(0.0, -Stot), eta, psi, pr[4], pr[7],
                                    sqrt(V[0] * V[0] + V[1] * V[1] + V[2] * V[2]));
      slips = true;
      ratio = mag > 0.0 ? (mag - eta * v) / mag : 1.0;
    } else {
      // below the strength the point is locked: tau = tau_lock, V = 0 exactly
      const double fr = mu_s - (mu_s - mu_d) * fmin(psi / dc, 1.0);
      const double strength = coh + fr * fmax(0.0, -Stot);
      slips = mag > strength;
      ratio = slips ? strength / mag : 1.0;
    }
    double speed2 = 0.0;
    for (int d = 0; d < 3; ++d) {
      Tb[d] = ratio * Ttot[d];
      const double tau = slips ? Tb[d] - tau0[d] : lock[d];
      V[d] = slips ? (lock[d] - tau) / eta : 0.0;
      speed2 += V[d] * V[d];
      atau[d] += wj * tau;
      avm[d] += wj * (vtm[d] + (tau - ttm[d]) / zsm);
      avp[d] += wj * (vtp[d] - (tau - ttp[d]) / zsp);
      slip[d] += wj * dt * V[d];
    }
    as += wj * s;
    avn += wj * vn;
    const double speed = sqrt(speed2);
    if (!rate_state) {
      psi += wj * dt * speed;
    } else if (speed > 0.0) {
      const double pss = rs_steady_state(speed, pr + 4);
      psi = pss + (psi - pss) * exp(-speed * wj * dt / pr[6]);
    }
  }
  for (int d = 0; d < 3; ++d) {
    st[d] = slip[d];
    st[4 + d] = V[d];
    st[7 + d] = Tb[d];
  }
  st[3] = psi;
  st[10] = Stot;
  // time-averaged middle states: stress s n n + tau n + n tau, velocity vn n + v_t
  double sig[6];
  sig[0] = as * n[0] * n[0] + 2.0 * atau[0] * n[0];
  sig[1] = as * n[1] * n[1] + 2.0 * atau[1] * n[1];
  sig[2] = as * n[2] * n[2] + 2.0 * atau[2] * n[2];
  sig[3] = as * n[0] * n[1] + atau[0] * n[1] + atau[1] * n[0];
  sig[4] = as * n[1] * n[2] + atau[1] * n[2] + atau[2] * n[1];
  sig[5] = as * n[0] * n[2] + atau[0] * n[2] + atau[2] * n[0];
  const int mr = a.pinv[h * Bf + m];
  for (int p = 0; p < 6; ++p) {
    In[inidx(em, fm, m, p, FT)] = (T)sig[p];
    In[inidx(ep, fp, mr, p, FT)] = (T)sig[p];
  }
  for (int d = 0; d < 3; ++d) {
    In[inidx(em, fm, m, 6 + d, FT)] = (T)(avn * n[d] + avm[d]);
    In[inidx(ep, fp, mr, 6 + d, FT)] = (T)(avn * n[d] + avp[d]);
  }
}

}  // namespace

template <typename T>
hipError_t launch_fault(int N, const FaultArgs& a, const T* gD, T* In, int64_t f0, int64_t nf, hipStream_t s) {
  if (nf <= 0) return hipSuccess;
  if (!a.elem || !a.face || !a.pelem || !a.pface || !a.perm || !a.geo || !a.par || !a.state || !a.Et || !a.pinv ||
      !a.dslot || !a.tq || !a.tw || !gD || !In)
    return hipErrorInvalidValue;
  switch (N) {
#define SEIS_F(NN) \
  case NN: hipLaunchKernelGGL((k_fault<T, NN>), dim3((unsigned)nf), dim3(kFaultThreads), 0, s, a, gD, In, f0); break;
    SEIS_F(1) SEIS_F(2) SEIS_F(3) SEIS_F(4) SEIS_F(5) SEIS_F(6)
#undef SEIS_F
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_fault<double>(int, const FaultArgs&, const double*, double*, int64_t, int64_t, hipStream_t);
template hipError_t launch_fault<float>(int, const FaultArgs&, const float*, float*, int64_t, int64_t, hipStream_t);

}  // namespace seis
