// The velocity-stress flux operator on the device.
//
// apply_A(e, v) = A_e v with A_x, A_y, A_z the Jacobians of
// q_t + A q_x + B q_y + C q_z = 0 (Sec. 3 PDE, Sec. 4.1 linear form), written
// out component by component (quantity order s_xx s_yy s_zz s_xy s_yz s_xz v_x v_y v_z).
// The scaled star matrix of an element is A*_d = sum_e G[d][e] A_e with
// G = dt * dxi/dx, so neither A_e nor A*_d is ever stored.
#pragma once

#include <hip/hip_runtime.h>

namespace seis {

// out_p = (sum_e c_e A_e) v for the combination c = (cx, cy, cz).
template <typename T>
__device__ __forceinline__ void apply_star(T cx, T cy, T cz, T lam, T mu, T rinv, const T v[9], T out[9]) {
  // the minus signs are carried by the coefficients: negation is exact, so
  // this equals -(l2m cx vx + ...) etc. bit for bit, without sign flips
  const T nl2m = -(lam + T(2) * mu), nlam = -lam, nmu = -mu, nr = -rinv;
  const T vx = v[6], vy = v[7], vz = v[8];
  out[0] = nl2m * cx * vx + nlam * cy * vy + nlam * cz * vz;
  out[1] = nlam * cx * vx + nl2m * cy * vy + nlam * cz * vz;
  out[2] = nlam * cx * vx + nlam * cy * vy + nl2m * cz * vz;
  out[3] = nmu * (cx * vy + cy * vx);
  out[4] = nmu * (cy * vz + cz * vy);
  out[5] = nmu * (cx * vz + cz * vx);
  out[6] = nr * (cx * v[0] + cy * v[3] + cz * v[5]);
  out[7] = nr * (cx * v[3] + cy * v[1] + cz * v[4]);
  out[8] = nr * (cx * v[5] + cy * v[4] + cz * v[2]);
}

// out_p = sum_e (A_e w_e)_p for three vectors w_x, w_y, w_z (physical gradient components).
template <typename T>
__device__ __forceinline__ T grad_op(int p, T lam, T mu, T rinv, const T* wx, const T* wy, const T* wz) {
  const T l2m = lam + T(2) * mu;
  switch (p) {
    case 0: return -(l2m * wx[6] + lam * wy[7] + lam * wz[8]);
    case 1: return -(lam * wx[6] + l2m * wy[7] + lam * wz[8]);
    case 2: return -(lam * wx[6] + lam * wy[7] + l2m * wz[8]);
    case 3: return -mu * (wx[7] + wy[6]);
    case 4: return -mu * (wy[8] + wz[7]);
    case 5: return -mu * (wx[8] + wz[6]);
    case 6: return -rinv * (wx[0] + wy[3] + wz[5]);
    case 7: return -rinv * (wx[3] + wy[1] + wz[4]);
    default: return -rinv * (wx[5] + wy[4] + wz[2]);
  }
}

// Minus the Godunov flux A-hat^-(n) q^b at one face node (Sec. 4.2), with the
// middle state a linear map of the given trace: c = n_x, n_y, n_z, then the
// eight scaled coefficients of (s_n^b, v_n^b) from (s_n, v_n) and
// (t_t^b, v_t^b) from (t_t, v_t).
template <typename T>
__device__ __forceinline__ void node_flux(const T* c, T lam, T mu, T rinv, const T* in, T* out) {
  const T nx = c[0], ny = c[1], nz = c[2];
  const T tx = in[0] * nx + in[3] * ny + in[5] * nz;
  const T ty = in[3] * nx + in[1] * ny + in[4] * nz;
  const T tz = in[5] * nx + in[4] * ny + in[2] * nz;
  const T sn = tx * nx + ty * ny + tz * nz;
  const T ttx = tx - sn * nx, tty = ty - sn * ny, ttz = tz - sn * nz;
  const T vn = in[6] * nx + in[7] * ny + in[8] * nz;
  const T vtx = in[6] - vn * nx, vty = in[7] - vn * ny, vtz = in[8] - vn * nz;
  const T snb = c[3] * sn + c[4] * vn;
  const T vnb = c[5] * sn + c[6] * vn;
  const T tbx = c[7] * ttx + c[8] * vtx, tby = c[7] * tty + c[8] * vty, tbz = c[7] * ttz + c[8] * vtz;
  const T vbx = c[9] * ttx + c[10] * vtx, vby = c[9] * tty + c[10] * vty, vbz = c[9] * ttz + c[10] * vtz;
  const T w = T(2) * vnb;
  // out is minus the flux (the sign every caller applies), so no sign flips
  out[0] = lam * vnb + mu * (w * nx * nx + T(2) * vbx * nx);
  out[1] = lam * vnb + mu * (w * ny * ny + T(2) * vby * ny);
  out[2] = lam * vnb + mu * (w * nz * nz + T(2) * vbz * nz);
  out[3] = mu * (w * nx * ny + vbx * ny + vby * nx);
  out[4] = mu * (w * ny * nz + vby * nz + vbz * ny);
  out[5] = mu * (w * nx * nz + vbx * nz + vbz * nx);
  out[6] = rinv * (snb * nx + tbx);
  out[7] = rinv * (snb * ny + tby);
  out[8] = rinv * (snb * nz + tbz);
}

__host__ __device__ constexpr int nbasis(int N) { return (N + 1) * (N + 2) * (N + 3) / 6; }
__host__ __device__ constexpr int nface(int N) { return (N + 1) * (N + 2) / 2; }

}  // namespace seis
