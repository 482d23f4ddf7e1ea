// Transposed Jacobians of the flux and of the Lax-Friedrichs flux, shared by
// the adjoint kernels (kern_vjp.hip, kern_vjp_line.hip).
#pragma once

#include "stage_fp64.h"

namespace dgdev {

// out += (dF^d/dQ)^T g at state q (Eq. (2) with the pressure of Eq. (3)).
template <int d>
__device__ __forceinline__ void flux_vjp(const double* q, const double* g, double gm1, double* out) {
  const double r = dgdev::recip(q[0]);
  const double u0 = q[1] * r, u1 = q[2] * r, u2 = q[3] * r;
  const double ud = d == 0 ? u0 : (d == 1 ? u1 : u2);
  const double pr = gm1 * (q[4] - 0.5 * (q[1] * u0 + q[2] * u1 + q[3] * u2));
  const double gd = d == 0 ? g[1] : (d == 1 ? g[2] : g[3]);
  // S = g0 m_d + sum_k g_k m_k u_d + g_d p + g4 (E + p) u_d
  const double B = g[1] * q[1] + g[2] * q[2] + g[3] * q[3] + g[4] * (q[4] + pr);  // dS/du_d
  const double P = gd + g[4] * ud;                                                // dS/dp
  const double usq = u0 * u0 + u1 * u1 + u2 * u2;
  out[0] += -B * ud * r + P * gm1 * 0.5 * usq;
  out[1] += g[1] * ud - P * gm1 * u0 + (d == 0 ? g[0] + B * r : 0.0);
  out[2] += g[2] * ud - P * gm1 * u1 + (d == 1 ? g[0] + B * r : 0.0);
  out[3] += g[3] * ud - P * gm1 * u2 + (d == 2 ? g[0] + B * r : 0.0);
  out[4] += g[4] * ud + P * gm1;
}

// Local wave speed l = |u_d| + c and its gradient dl/dq.
template <int d>
__device__ __forceinline__ double wave_speed_grad(const double* q, double gamma, double gm1, double* dl) {
  const double r = dgdev::recip(q[0]);
  const double u0 = q[1] * r, u1 = q[2] * r, u2 = q[3] * r;
  const double ud = d == 0 ? u0 : (d == 1 ? u1 : u2);
  const double usq = u0 * u0 + u1 * u1 + u2 * u2;
  const double e = gm1 * (q[4] * r - 0.5 * usq);  // p / rho
  const double c = dgdev::root(gamma * e);
  const double sg = ud >= 0.0 ? 1.0 : -1.0;
  const double k = gamma * dgdev::recip(2.0 * c);
  // de/drho = gm1 (-E/rho + |u|^2)/rho, de/dm_k = -gm1 u_k / rho, de/dE = gm1 / rho
  dl[0] = sg * (-ud * r) + k * gm1 * (-q[4] * r + usq) * r;
  dl[1] = (d == 0 ? sg * r : 0.0) - k * gm1 * u0 * r;
  dl[2] = (d == 1 ? sg * r : 0.0) - k * gm1 * u1 * r;
  dl[3] = (d == 2 ? sg * r : 0.0) - k * gm1 * u2 * r;
  dl[4] = k * gm1 * r;
  return fabs(ud) + c;
}

// Transpose of the local Lax-Friedrichs Jacobian for one side, applied to g:
// minus side:  (1/2) A(qm)^T g + (lambda/2) g - (1/2)(g . (qp - qm)) dlambda/dqm
// plus side:   (1/2) A(qp)^T g - (lambda/2) g - (1/2)(g . (qp - qm)) dlambda/dqp
template <int d>
__device__ __forceinline__ void lf_vjp_d(const double* qm, const double* qp, double gamma, double gm1,
                                         const double* g, bool minus_side, double* out) {
  double dlm[5], dlp[5];
  const double lm = wave_speed_grad<d>(qm, gamma, gm1, dlm);
  const double lp = wave_speed_grad<d>(qp, gamma, gm1, dlp);
  const bool pick_m = lm >= lp;
  const double lam = pick_m ? lm : lp;
  double gdel = 0.0;
#pragma unroll
  for (int f = 0; f < 5; ++f) gdel += g[f] * (qp[f] - qm[f]);
  double hg[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    hg[f] = 0.5 * g[f];
    out[f] = 0.0;
  }
  double qs[5], dl[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    qs[f] = minus_side ? qm[f] : qp[f];
    dl[f] = minus_side ? dlm[f] : dlp[f];
  }
  flux_vjp<d>(qs, hg, gm1, out);
  const bool own_selected = minus_side ? pick_m : !pick_m;
  const double sl = minus_side ? 0.5 * lam : -0.5 * lam;
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    out[f] += sl * g[f];
    if (own_selected) out[f] -= 0.5 * gdel * dl[f];
  }
}

}  // namespace dgdev
