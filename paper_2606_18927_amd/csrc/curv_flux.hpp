// Fluxes on curvilinear elements: two-point and Roe fluxes contracted with a metric
// vector, viscous stress and contravariant viscous flux.
#pragma once

#include "dg_device.hpp"

namespace dg {
namespace {

// Chandrashekar's flux contracted with the metric vector M (the average of the
// two nodes' J a^i in the volume, the face normal on a face): with
// a, b = (rho, u, v, w, beta, |u|^2), beta = rho / (2 p), U~ = {{u}} . M,
//   F_rho = rho_ln U~,  F_m = F_rho {{u}} + p^ M,  p^ = {{rho}} / (2 {{beta}}),
//   F_E = F_rho (1 / (2 (gamma - 1) beta_ln) - {{|u|^2}} / 2) + {{u}} . F_m.
__device__ inline void ec_flux_contra(const double a[6], const double b[6], double M0, double M1, double M2,
                                      double gm1, double f[5]) {
  double rho_ln, inv_beta_ln, p_hat;
  ec_means(a[0], b[0], a[4], b[4], rho_ln, inv_beta_ln, p_hat);
  const double u = 0.5 * (a[1] + b[1]), v = 0.5 * (a[2] + b[2]), w = 0.5 * (a[3] + b[3]);
  const double q2 = 0.5 * (a[5] + b[5]);
  const double F1 = rho_ln * (u * M0 + v * M1 + w * M2);
  f[0] = F1;
  f[1] = F1 * u + p_hat * M0;
  f[2] = F1 * v + p_hat * M1;
  f[3] = F1 * w + p_hat * M2;
  f[4] = F1 * (0.5 / gm1 * inv_beta_ln - 0.5 * q2) + f[1] * u + f[2] * v + f[3] * w;
}

// Roe's dissipation sum_k |lambda_k| alpha_k r_k across a face with unit
// normal n (L on the side n points away from; primitives (rho, u, v, w, p)
// and total energies E), linearised at the Roe average (sqrt(rho)-weighted u
// and H = (E + p) / rho, rho~ = sqrt(rho_L rho_R), a~^2 = (gamma - 1)(H~ - |u~|^2/2)):
// acoustic waves u~.n -+ a~ with alpha = ([[p]] -+ rho~ a~ [[u.n]]) / (2 a~^2),
// r = (1, u~ -+ a~ n, H~ -+ (u~.n) a~) and Harten-Hyman |lambda|; the entropy
// wave u~.n with alpha = [[rho]] - [[p]] / a~^2, r = (1, u~, |u~|^2 / 2); the
// shear wave u~.n with rho~ (0, [[u]]_t, u~ . [[u]]_t), [[u]]_t = [[u]] - [[u.n]] n.
__device__ inline void roe_dissipation_normal(const double L[5], double EL, const double R[5], double ER,
                                              const double n[3], double gamma, double D[5]) {
  const double sl = sqrt_nr(L[0]), sr = sqrt_nr(R[0]);
  const double iL = rcp_nr(L[0]), iR = rcp_nr(R[0]);
  const double isum = rcp_nr(sl + sr);
  const double wl = sl * isum, wr = sr * isum;
  double ut[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) ut[c] = wl * L[1 + c] + wr * R[1 + c];
  const double H = quot(wl * (EL + L[4]), L[0], iL) + quot(wr * (ER + R[4]), R[0], iR);
  const double q2 = ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2];
  const double a2 = (gamma - 1.0) * (H - 0.5 * q2);
  const double a = sqrt_nr(a2), ia2 = rcp_nr(a2);
  const double rho = sl * sr;
  const double un = ut[0] * n[0] + ut[1] * n[1] + ut[2] * n[2];
  const double dp = R[4] - L[4];
  double du[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) du[c] = R[1 + c] - L[1 + c];
  const double dun = du[0] * n[0] + du[1] * n[1] + du[2] * n[2];
  const double al1 = 0.5 * quot(dp - rho * a * dun, a2, ia2);
  const double al5 = 0.5 * quot(dp + rho * a * dun, a2, ia2);
  const double al2 = (R[0] - L[0]) - quot(dp, a2, ia2);
  const double unl = L[1] * n[0] + L[2] * n[1] + L[3] * n[2], unr = R[1] * n[0] + R[2] * n[1] + R[3] * n[2];
  const double cl = sqrt_nr(quot(gamma * L[4], L[0], iL)), cr = sqrt_nr(quot(gamma * R[4], R[0], iR));
  const double l1 = hh_abs(un - a, unl - cl, unr - cr);
  const double l5 = hh_abs(un + a, unl + cl, unr + cr);
  const double l2 = fabs(un);
  const double t1 = l1 * al1, t5 = l5 * al5, t2 = l2 * al2, ts = l2 * rho;
  double udt = 0.0;
  D[0] = t1 + t2 + t5;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double sh = du[c] - dun * n[c];
    udt += ut[c] * sh;
    D[1 + c] = (t1 + t2 + t5) * ut[c] + (t5 - t1) * a * n[c] + ts * sh;
  }
  D[4] = t1 * (H - un * a) + t2 * (0.5 * q2) + t5 * (H + un * a) + ts * udt;
}

// Own-side contravariant viscous flux along metric vector M from the stress:
// (sum_d M_d tau_0d, sum_d M_d tau_1d, sum_d M_d tau_2d, u . (those) + M . qT)
template <typename R>
__device__ inline void contra_viscous(R u, R v, R w, const R tau[6], const R qT[3], R M0, R M1, R M2,
                                      R f[4]) {
  f[0] = M0 * tau[0] + M1 * tau[3] + M2 * tau[4];
  f[1] = M0 * tau[3] + M1 * tau[1] + M2 * tau[5];
  f[2] = M0 * tau[4] + M1 * tau[5] + M2 * tau[2];
  f[3] = u * f[0] + v * f[1] + w * f[2] + M0 * qT[0] + M1 * qT[1] + M2 * qT[2];
}

// Stress (t00, t11, t22, t01, t02, t12) and heat flux of physical gradients g[3 q + d]
template <typename R>
__device__ inline void stress64(const R g[12], R mu, R kappa, R tau[6], R qT[3]) {
  const R dd = R(2.0 / 3.0) * (g[0] + g[4] + g[8]);
  tau[0] = mu * (g[0] + g[0] - dd);
  tau[1] = mu * (g[4] + g[4] - dd);
  tau[2] = mu * (g[8] + g[8] - dd);
  tau[3] = mu * (g[1] + g[3]);
  tau[4] = mu * (g[2] + g[6]);
  tau[5] = mu * (g[5] + g[7]);
  qT[0] = kappa * g[9];
  qT[1] = kappa * g[10];
  qT[2] = kappa * g[11];
}

}  // namespace
}  // namespace dg
