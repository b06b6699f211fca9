// Vector-Jacobian product (adjoint) of the DGSEM right-hand side, FP64.
//
// Ubar = (dL/dU)^T lam is evaluated as a gather: every element computes the
// cotangent of its own nodal state and pulls what its neighbours' equations
// contribute through shared face nodes, so no atomics are needed and the
// result is deterministic.  Two kernels:
//
//   k_vjp_a : lam (+ neighbour lam at face nodes), U ->
//             the forward BR1 gradients of U (recomputed in LDS, as in the
//             forward right-hand side), then
//             gbar = cotangent of the lifted gradients (12 per node) and the
//             part of Ubar that does not pass through the lifting.  In the weak form
//             (line_device.hpp), with Q = diag(w) D and l_i = s_d lam_i / w_i:
//               * volume split form: for each line pair i < m, both nodes take
//                 J1^T (-2 Q_im (l_i - l_m)), J1 = d f#(a, b) / d a of the symmetric
//                 two-point flux (Kennedy-Gruber, or Chandrashekar's with its
//                 logarithmic means differentiated on the branch the forward takes);
//               * viscous volume term: Fvbar_d = -(weak derivative of l, the
//                 neighbours' l as ghosts), then the transpose of
//                 f_v,d(u, grad) -> (ubar, gbar);
//               * each face node's numerical flux, which enters both sides'
//                 equations, with the combined cotangent phi = -+(l_o - l_n) (the own
//                 physical flux cancels with the diagonal of the volume sum);
//               * the primitive map P(U) transposed.
//   k_vjp_b : gbar (+ neighbour gbar at face nodes) -> qbar of q = (u, v, w, T)
//             through the transposed BR1 lifting, then Ubar += (dq/dU)^T qbar.
//
// The Roe dissipation's derivative is written out in reverse mode.  Non-smooth
// points: |u_d| and the max of the Lax-Friedrichs speed, and |lambda| and the
// entropy correction's branch of the Roe flux, take the derivative of the
// branch that is active (ties to the lower side L), as the CPU oracle's
// reverse mode does.
#include "line_device.hpp"

namespace dg {
namespace {

// abar += (d f#(a, b) / d a)^T mu, a and b primitive (rho, u, v, w, p, e), u along the line.
__device__ inline void kg_vjp(const double a[6], const double b[6], const double mu[5],
                              double abar[6]) {
  const double rho = 0.5 * (a[0] + b[0]);
  const double u0 = 0.5 * (a[1] + b[1]), u1 = 0.5 * (a[2] + b[2]), u2 = 0.5 * (a[3] + b[3]);
  const double p = 0.5 * (a[4] + b[4]);
  const double e = 0.5 * (a[5] + b[5]);
  const double mass = rho * u0;
  const double S = mu[0] + u0 * mu[1] + u1 * mu[2] + u2 * mu[3] + e * mu[4];
  abar[0] += 0.5 * u0 * S;
  abar[1] += 0.5 * mass * mu[1];
  abar[2] += 0.5 * mass * mu[2];
  abar[3] += 0.5 * mass * mu[3];
  abar[1] += 0.5 * (rho * S + p * mu[4]);
  abar[4] += 0.5 * (mu[1] + u0 * mu[4]);
  abar[5] += 0.5 * mass * mu[4];
}

// Ubar += (dP/dU)^T Pbar + (dT/dU)^T Tbar at the primitives P = (rho, u, v, w, p, e),
// T = p/(rho R).  P are the values that the fluxes were transposed at: the terms in e of
// rho's cotangent, hundreds of velocities squared at Ma = 0.1, cancel between the pairs and
// here only for the same e (with e formed again from rho e: 2.5 times the rounding error).
__device__ inline void prim_vjp(const double P[6], const double Pb[6], double Tb, const DevPhys& ph, double Ub[5]) {
  const double ir = 1.0 / P[0];
  const double u = P[1], v = P[2], w = P[3], e = P[5];
  const double q2 = u * u + v * v + w * w;
  const double T = P[4] * ph.inv_R * ir;
  const double pb = Pb[4] + Tb * ir * ph.inv_R;
  const double rb = Pb[0] - Tb * T * ir;
  Ub[0] += rb - ir * (u * Pb[1] + v * Pb[2] + w * Pb[3]) + 0.5 * ph.gm1 * q2 * pb - e * ir * Pb[5];
  Ub[1] += ir * Pb[1] - ph.gm1 * u * pb;
  Ub[2] += ir * Pb[2] - ph.gm1 * v * pb;
  Ub[3] += ir * Pb[3] - ph.gm1 * w * pb;
  Ub[4] += ph.gm1 * pb + ir * Pb[5];
}

// abar += lb d(|u| + c)/dP, c = sqrt(gamma p / rho).
__device__ inline void speed_vjp(const double a[6], double lb, const DevPhys& ph, double abar[6]) {
  const double c = sqrt(ph.gamma * a[4] / a[0]);
  const double ud = a[1];
  abar[1] += lb * (ud > 0.0 ? 1.0 : (ud < 0.0 ? -1.0 : 0.0));
  abar[4] += lb * 0.5 * c / a[4];
  abar[0] -= lb * 0.5 * c / a[0];
}

__device__ inline void to_prim(const double s[5], const DevPhys& ph, double a[6]) {
  const Prim P = primitives(s, ph);
  a[0] = P.rho;
  a[1] = P.u;
  a[2] = P.v;
  a[3] = P.w;
  a[4] = P.p;
  a[5] = P.e;
}

// ---- entropy-conserving / Roe pair ----

// Logarithmic-mean factors of f = (x_a - x_b) / (x_a + x_b) (the forward
// pair's switch: series for f^2 < 1e-4, atanh otherwise):
//   G = f / atanh f (x_ln = (x_a + x_b) G / 2),  F = atanh f / f (1 / x_ln = 2 F / (x_a + x_b)),
// with dG = dG/df and dF = dF/df.
__device__ inline void ln_mean_factors(double f, double& G, double& dG, double& F, double& dF,
                                       bool want_G) {
  const double u = f * f;
  if (u < 1e-4) {
    G = 1.0 - u * (1.0 / 3.0 + u * (4.0 / 45.0 + u * (44.0 / 945.0)));
    dG = -2.0 * f * (1.0 / 3.0 + u * (8.0 / 45.0 + u * (132.0 / 945.0)));
    F = 1.0 + u * (1.0 / 3.0 + u * (0.2 + u * (1.0 / 7.0)));
    dF = 2.0 * f * (1.0 / 3.0 + u * (0.4 + u * (3.0 / 7.0)));
  } else {
    const double t = atanh(f), r = f / (1.0 - u);
    if (want_G) {
      G = f / t;
      dG = (t - r) / (t * t);
    } else {
      F = t / f;
      dF = (r - t) / u;
    }
  }
}

// abar += (d f#_EC(a, b) / d a)^T mu for Chandrashekar's flux along the line, a and b
// = (rho, u, v, w, p, beta), beta = rho / (2 p); abar[5] is the cotangent of
// beta (p enters the flux only through beta).  With um = {{u}},
// q2m = {{|u|^2}}, F1 = rho_ln um_0, p^ = {{rho}} / (2 {{beta}}) and
// kappa = 1 / (2 (gamma - 1)), mu . f# = F1 A + p^ Bp where
//   A = mu_0 + mu_m . um + mu_4 (kappa / beta_ln - q2m / 2 + |um|^2),  Bp = mu_1 + mu_4 um_0.
__device__ inline void ec_vjp(const double a[6], const double b[6], const double mu[5],
                              double gm1, double abar[6]) {
  const double sr = a[0] + b[0], sb = a[5] + b[5];
  const double ir = 1.0 / sr, ib = 1.0 / sb;
  double G, dG, F, dF, unused0, unused1;
  ln_mean_factors((a[0] - b[0]) * ir, G, dG, unused0, unused1, true);
  ln_mean_factors((a[5] - b[5]) * ib, unused0, unused1, F, dF, false);
  const double rho_ln = 0.5 * sr * G;
  const double ibl = 2.0 * ib * F;
  const double p_hat = 0.5 * sr * ib;
  const double um[3] = {0.5 * (a[1] + b[1]), 0.5 * (a[2] + b[2]), 0.5 * (a[3] + b[3])};
  const double q2m = 0.5 * (a[1] * a[1] + a[2] * a[2] + a[3] * a[3] + b[1] * b[1] + b[2] * b[2] + b[3] * b[3]);
  const double um2 = um[0] * um[0] + um[1] * um[1] + um[2] * um[2];
  const double F1 = rho_ln * um[0];
  const double kap = 0.5 / gm1;
  const double A = mu[0] + mu[1] * um[0] + mu[2] * um[1] + mu[3] * um[2] +
                   mu[4] * (kap * ibl - 0.5 * q2m + um2);
  const double Bp = mu[1] + mu[4] * um[0];
  // d rho_ln / d rho_a = G / 2 + rho_b G' / sr;  d (1 / beta_ln) / d beta_a = -2 ib^2 F + 4 beta_b ib^3 F'
  const double drl = 0.5 * G + b[0] * dG * ir;
  const double dibl = ib * ib * (-2.0 * F + 4.0 * b[5] * ib * dF);
  abar[0] += A * um[0] * drl + 0.5 * ib * Bp;
  abar[5] += F1 * mu[4] * kap * dibl - 0.5 * sr * ib * ib * Bp;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double sk = F1 * (mu[1 + k] + 2.0 * mu[4] * um[k]);
    if (k == 0) sk += mu[4] * p_hat + A * rho_ln;
    abar[1 + k] += 0.5 * sk - 0.5 * F1 * mu[4] * a[1 + k];
  }
}

// Pb += the (rho, u, v, w, p) cotangent of Pbe, whose slot 5 is the cotangent
// of beta = rho / (2 p) at the primitives a.
__device__ inline void fold_beta(const double a[6], const double Pbe[6], double Pb[6]) {
  const double ip = 1.0 / a[4];
#pragma unroll
  for (int q = 0; q < 5; ++q) Pb[q] += Pbe[q];
  Pb[0] += 0.5 * ip * Pbe[5];
  Pb[4] -= a[5] * ip * Pbe[5];
}

// lam_bar, lamL_bar, lamR_bar += gb d hh(lam, lamL, lamR): Harten-Hyman |lambda|
// (the branch and the max that the values select, ties to the first argument).
__device__ inline void hh_vjp(double lam, double lamL, double lamR, double gb, double& lb,
                              double& lLb, double& lRb) {
  const double d1 = lam - lamL, d2 = lamR - lam;
  const bool first = d1 >= d2;
  const double delta = first ? d1 : d2;
  if (delta > 0.0 && fabs(lam) < delta) {
    const double bd = gb * (delta * delta - lam * lam) / (2.0 * delta * delta);
    lb += gb * lam / delta + (first ? bd : -bd);
    if (first)
      lLb -= bd;
    else
      lRb += bd;
  } else {
    lb += lam > 0.0 ? gb : (lam < 0.0 ? -gb : 0.0);
  }
}

// Pb += -(1/2) (d Roe(U_L, U_R) / d P_own)^T phi in the own primitives
// (rho, u, v, w, p, e): reverse mode of the Roe dissipation (the forward
// quantities of that function, then their cotangents in reverse order), own =
// L when own_L; E = rho e carries the total-energy cotangent into rho and e.
__device__ inline void roe_vjp(const double so[5], const double sn[5], bool own_L,
                               const double phi[5], const DevPhys& ph, double Pb[6]) {
  const double* sL = own_L ? so : sn;
  const double* sR = own_L ? sn : so;
  double L[5], R[5];
  {
    const double il = 1.0 / sL[0], ir = 1.0 / sR[0];
    L[0] = sL[0];
    R[0] = sR[0];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      L[1 + c] = sL[1 + c] * il;
      R[1 + c] = sR[1 + c] * ir;
    }
    L[4] = ph.gm1 * (sL[4] - 0.5 * sL[0] * (L[1] * L[1] + L[2] * L[2] + L[3] * L[3]));
    R[4] = ph.gm1 * (sR[4] - 0.5 * sR[0] * (R[1] * R[1] + R[2] * R[2] + R[3] * R[3]));
  }
  const double EL = sL[4], ER = sR[4];
  // forward
  const double sl = sqrt(L[0]), sr = sqrt(R[0]);
  const double isum = 1.0 / (sl + sr);
  const double wl = sl * isum, wr = sr * isum;
  double ut[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) ut[c] = wl * L[1 + c] + wr * R[1 + c];
  const double hL = (EL + L[4]) / L[0], hR = (ER + R[4]) / R[0];
  const double H = wl * hL + wr * hR;
  const double q2 = ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2];
  const double a2 = ph.gm1 * (H - 0.5 * q2);
  const double a = sqrt(a2);
  const double rho = sl * sr;
  const double un = ut[0];
  const double dp = R[4] - L[4];
  const double dud = R[1] - L[1];
  const double i2a2 = 0.5 / a2;
  const double al1 = (dp - rho * a * dud) * i2a2, al5 = (dp + rho * a * dud) * i2a2;
  const double al2 = (R[0] - L[0]) - dp / a2;
  const double cl = sqrt(ph.gamma * L[4] / L[0]), cr = sqrt(ph.gamma * R[4] / R[0]);
  const double l1 = hh_abs(un - a, L[1] - cl, R[1] - cr);
  const double l5 = hh_abs(un + a, L[1] + cl, R[1] + cr);
  const double l2 = fabs(un);
  const double t1 = l1 * al1, t5 = l5 * al5, t2 = l2 * al2, ts = l2 * rho;
  const double T = t1 + t2 + t5;
  // reverse, with the cotangent -phi/2 of the dissipation
  double g[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) g[v] = -0.5 * phi[v];
  double Lb[5] = {0, 0, 0, 0, 0}, Rb[5] = {0, 0, 0, 0, 0};
  double Tb = g[0], tsb = 0.0, udtb = g[4] * ts, utb[3], udt = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double sh = c == 0 ? 0.0 : R[1 + c] - L[1 + c];
    udt += ut[c] * sh;
    Tb += g[1 + c] * ut[c];
    utb[c] = g[1 + c] * T + udtb * sh;
    tsb += g[1 + c] * sh;
    // the shear jump (c != 0): ts d(D_{1+c})/d du_c + ut_c d(D_4)/d du_c
    const double dub = c == 0 ? 0.0 : g[1 + c] * ts + udtb * ut[c];
    Rb[1 + c] += dub;
    Lb[1 + c] -= dub;
  }
  double t5b = g[1] * a + g[4] * (H + un * a) + Tb;
  double t1b = -g[1] * a + g[4] * (H - un * a) + Tb;
  const double t2b = g[4] * 0.5 * q2 + Tb;
  tsb += g[4] * udt;
  double ab = (g[1] + g[4] * un) * (t5 - t1);
  double Hb = g[4] * (t1 + t5);
  double unb = g[4] * a * (t5 - t1);
  double q2b = g[4] * 0.5 * t2;
  const double l2b = tsb * rho + t2b * al2;
  double rhob = tsb * l2;
  const double al2b = t2b * l2, al5b = t5b * l5, al1b = t1b * l1;
  unb += un > 0.0 ? l2b : (un < 0.0 ? -l2b : 0.0);
  double b5 = 0.0, bL5 = 0.0, bR5 = 0.0, b1 = 0.0, bL1 = 0.0, bR1 = 0.0;
  hh_vjp(un + a, L[1] + cl, R[1] + cr, t5b * al5, b5, bL5, bR5);
  hh_vjp(un - a, L[1] - cl, R[1] - cr, t1b * al1, b1, bL1, bR1);
  unb += b5 + b1;
  ab += b5 - b1;
  Lb[1] += bL5 + bL1;
  Rb[1] += bR5 + bR1;
  const double clb = bL5 - bL1, crb = bR5 - bR1;
  Lb[4] += clb * cl / (2.0 * L[4]);
  Lb[0] -= clb * cl / (2.0 * L[0]);
  Rb[4] += crb * cr / (2.0 * R[4]);
  Rb[0] -= crb * cr / (2.0 * R[0]);
  Rb[0] += al2b;
  Lb[0] -= al2b;
  const double dpb = -al2b / a2 + (al1b + al5b) * i2a2;
  double a2b = al2b * dp / (a2 * a2) - (al1b * al1 + al5b * al5) / a2;
  const double dal = (al5b - al1b) * i2a2;
  rhob += dal * a * dud;
  ab += dal * rho * dud;
  const double dudb = dal * rho * a;
  Rb[1] += dudb;
  Lb[1] -= dudb;
  Rb[4] += dpb;
  Lb[4] -= dpb;
  utb[0] += unb;
  double slb = rhob * sr, srb = rhob * sl;
  a2b += ab / (2.0 * a);
  Hb += a2b * ph.gm1;
  q2b -= 0.5 * a2b * ph.gm1;
  double wlb = Hb * hL, wrb = Hb * hR;
  const double hLb = Hb * wl, hRb = Hb * wr;
  const double ELb = hLb / L[0], ERb = hRb / R[0];
  Lb[4] += ELb;
  Lb[0] -= ELb * hL;
  Rb[4] += ERb;
  Rb[0] -= ERb * hR;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double u_b = utb[c] + 2.0 * q2b * ut[c];
    wlb += u_b * L[1 + c];
    wrb += u_b * R[1 + c];
    Lb[1 + c] += u_b * wl;
    Rb[1 + c] += u_b * wr;
  }
  slb += (wlb - wrb) * sr * isum * isum;
  srb += (wrb - wlb) * sl * isum * isum;
  Lb[0] += slb / (2.0 * sl);
  Rb[0] += srb / (2.0 * sr);
  // the own side: (rho, u, v, w, p) and E = rho e
  const double* Xb = own_L ? Lb : Rb;
  const double Eb = own_L ? ELb : ERb;
#pragma unroll
  for (int q = 0; q < 5; ++q) Pb[q] += Xb[q];
  Pb[0] += Eb * so[4] / so[0];
  Pb[5] += Eb * so[0];
}

// Scale s_d of the neighbour across face (d, up) of element (ex, ey, ez).
__device__ inline double nb_scale(const DevMesh& m, int ex, int ey, int ez, int d, bool up) {
  const int c = d == 0 ? ex : (d == 1 ? ey : ez);
  int v = c + (up ? 1 : -1);
  if (v < 0) v = m.n[d] - 1;
  if (v >= m.n[d]) v = 0;
  return m.s[d][v];
}

// --------------------------------------------------------------------------
// k_vjp_a
// --------------------------------------------------------------------------
struct VjpArgs {
  const double* U;
  const double* lam;
  double* gbar;
  double* ubar;
  DevMesh mesh;
  DevPhys ph;
  DevBasis basis;
};
typedef const __attribute__((address_space(4))) VjpArgs* VjpArgsPtr;

__device__ inline const VjpArgs& again(VjpArgsPtr p) {
  asm volatile("" : "+s"(p));
  return *(const VjpArgs*)p;
}

// One workgroup per element: LW waves of line lanes (the pairs of a line) and as many
// of face lanes (the faces at the line's ends and all its derivatives); a node
// phase takes one node per lane.  LDS fields (of EB values): halves of rho, u, v, w, p, e
// (entropy-conserving pair: beta in place of p), T, lam (5); raw gradients GR + 3 q + d;
// viscous flux cotangents FV + 3 c + d.  At the end the lines' sums (6 per direction) take
// the place of the latter two, the faces' cotangents END that of T and lam.
//
// What bounds it (N = 5, 48 x 32 x 48 elements, Kennedy-Gruber pair: 1.35 ms in reverse RK
// steps, 1.40 in single calls; with one lane per node 1.62, 1.80): 4.1 GB of HBM traffic
// (0.64 ms for a triad), vector instructions issue 57 % of the time (405 M wave
// instructions), LDS is busy 41 %, and the neighbours' values
// at the line ends (20 loads per face lane, each of 64 addresses in as many cache
// lines) hold up both.  Without the pairs it is 1.5 % faster, without the stores of
// gbar 10 %.  A second load of the neighbours' lam by the line lanes cost 0.08 ms, three
// workgroups per CU instead of two (24 fields, pairs in blocks) 0.13, workgroups that
// loop over elements and fetch the next one early 0.2.
// The same shape at the other degrees (us per transposed right-hand side, both kernels; with
// one lane per node in brackets; entropy-conserving pair with density noise of 0.1 / 5 / 40 %):
//   N = 3, 32^3, 128 lanes for 64 nodes          291 (345)   445 / 509 / 599 (612 / 1037 / 1036)
//   N = 5, 24^3                                  402 (451)   481 / 597 / 958 (774 / 1493 / 1494)
//   N = 7, 16^3, 147 KB LDS, one workgroup a CU  294 (378)   398 / 486 / 771 (553 / 1093 / 1092)
template <int N>
struct VjpShape {
  using L = Line<N>;
  static constexpr int LW = L::LW, BS = N == 7 ? 512 : 128 * LW;
  static constexpr int T = 6, LAM = 7, GR = 12, FV = 24, SUM = 12;
  static constexpr int END = 6 * L::EB >= 10 * L::LINES ? T * L::EB : 36 * L::EB;
  static constexpr int HEAD = 8;  // 1 / w_i
  static constexpr size_t BYTES = 8 * (HEAD + 36 * L::EB + (END == 36 * L::EB ? 10 * L::LINES : 0));
  static constexpr int BLOCK = N == 7 ? 4 : L::NP;  // nodes of a line held in registers
};

// dF/df of F = atanh f / f for u = f^2 below 1e-2 (dropped terms below 1e-16).
__device__ inline double ln_series_slope(double f, double u) {
  return 2.0 * f * (1.0 / 3.0 + u * (2.0 / 5.0 + u * (3.0 / 7.0 + u * (4.0 / 9.0 + u * (5.0 / 11.0 + u * (6.0 / 13.0 + u * (7.0 / 15.0 + u * (8.0 / 17.0))))))));
}

// The node of the pair sums: what a line lane reads of node m, x = (rho, u, v, w) / 2 in
// the line frame, then (p, e) / 2 or (beta, |u|^2 / 4), and lam c / w_m (c = -s_d, or -2 s_d).
template <int N, bool EC>
__device__ __forceinline__ void vjp_node(const double* sF, const double* inv_w, const LineTask<N>& t, int m, double c,
                                         double (&x)[11]) {
  using S = VjpShape<N>;
  constexpr int EB = Line<N>::EB;
  const int l = t.node(m);
  x[0] = sF[l];
  x[1] = sF[(1 + t.d) * EB + l];
  x[2] = sF[(1 + t.d1) * EB + l];
  x[3] = sF[(1 + t.d2) * EB + l];
  x[4] = sF[4 * EB + l];
  x[5] = EC ? x[1] * x[1] + x[2] * x[2] + x[3] * x[3] : sF[5 * EB + l];
  const double f = c * inv_w[m];
  x[6] = f * sF[S::LAM * EB + l];
  x[7] = f * sF[(S::LAM + 1 + t.d) * EB + l];
  x[8] = f * sF[(S::LAM + 1 + t.d1) * EB + l];
  x[9] = f * sF[(S::LAM + 1 + t.d2) * EB + l];
  x[10] = f * sF[(S::LAM + 4) * EB + l];
}

// One Kennedy-Gruber pair, cotangent mu = Q_im (lam_i / w_i - lam_m / w_m) (-2 s_d)
// on f#(i, m) (half of it here, for the means).  f# depends on sums only, so both nodes
// take the same increments; with S = mu_0 + u . mu_m + e mu_4 and m = rho u_d
//   (u_d S, m mu_m + e_d (rho S + p mu_4), mu_d + u_d mu_4, m mu_4).
__device__ __forceinline__ void kg_pair_vjp(const double (&a)[11], const double (&b)[11], double q, double (&ya)[6],
                                            double (&yb)[6]) {
  const double rho = a[0] + b[0], u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3], p = a[4] + b[4], e = a[5] + b[5];
  const double m0 = q * (a[6] - b[6]), m1 = q * (a[7] - b[7]), m2 = q * (a[8] - b[8]), m3 = q * (a[9] - b[9]),
               m4 = q * (a[10] - b[10]);
  const double S = m0 + u * m1 + v * m2 + w * m3 + e * m4;
  const double m = rho * u;
  const double du = m * m1 + rho * S + p * m4, dp = m1 + u * m4;
  ya[0] += u * S;
  yb[0] += u * S;
  ya[1] += du;
  yb[1] += du;
  ya[2] += m * m2;
  yb[2] += m * m2;
  ya[3] += m * m3;
  yb[3] += m * m3;
  ya[4] += dp;
  yb[4] += dp;
  ya[5] += m * m4;
  yb[5] += m * m4;
}

// One entropy-conserving pair (ec_vjp for both nodes at once): y[4] is the cotangent of
// beta.  MEANS: the logarithmic means' factors by the short series (f^2 below 1e-4), the
// long one (1e-2), or chosen pair by pair.
template <int MEANS>
__device__ __forceinline__ void ec_pair_vjp(const double (&a)[11], const double (&b)[11], double q, double kap,
                                            double (&ya)[6], double (&yb)[6]) {
  const double sr = a[0] + b[0], sb = a[4] + b[4];  // {{rho}}, 2 {{beta}}
  const double x = rcp_nr(sr * sb);
  const double ir = sb * x, ib = sr * x;
  const double fr = (a[0] - b[0]) * ir, fb = (a[4] - b[4]) * ib;
  const double ur = fr * fr, ub = fb * fb;
  double G, dG, F, dF;
  if constexpr (MEANS == 0) {
    G = 1.0 - ur * (1.0 / 3.0 + ur * (4.0 / 45.0 + ur * (44.0 / 945.0)));
    dG = -2.0 * fr * (1.0 / 3.0 + ur * (8.0 / 45.0 + ur * (132.0 / 945.0)));
    F = 1.0 + ub * (1.0 / 3.0 + ub * (0.2 + ub * (1.0 / 7.0)));
    dF = 2.0 * fb * (1.0 / 3.0 + ub * (0.4 + ub * (3.0 / 7.0)));
  } else if constexpr (MEANS == 1) {
    double unused;
    ln_series(ur, unused, G);
    dG = -ln_series_slope(fr, ur) * (G * G);
    ln_series(ub, F, unused);
    dF = ln_series_slope(fb, ub);
  } else {
    double unused0, unused1;
    ln_mean_factors(fr, G, dG, unused0, unused1, true);
    ln_mean_factors(fb, unused0, unused1, F, dF, false);
  }
  const double m0 = q * (a[6] - b[6]), m1 = q * (a[7] - b[7]), m2 = q * (a[8] - b[8]), m3 = q * (a[9] - b[9]),
               m4 = q * (a[10] - b[10]);
  const double u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3];
  const double rho_ln = sr * G, p_hat = sr * ib, F1 = rho_ln * u;
  const double A = m0 + m1 * u + m2 * v + m3 * w +
                   m4 * (2.0 * kap * ib * F - (a[5] + b[5]) + (u * u + v * v + w * w));
  const double Bp = m1 + m4 * u, hb = 0.5 * ib * Bp;
  // d rho_ln / d rho_a = G / 2 + rho_b G' / (2 {{rho}}), and of b with G' odd
  const double Au = A * u, Ag = 0.5 * Au * G + hb, At = Au * dG * ir;
  ya[0] += Ag + b[0] * At;
  yb[0] += Ag - a[0] * At;
  // d (1 / beta_ln) / d beta_a = ib^2 (-2 F + 4 beta_b ib F')
  const double k5 = F1 * m4 * kap * ib * ib;
  const double c5 = -2.0 * k5 * F - p_hat * ib * Bp, t5 = 4.0 * k5 * ib * dF;
  ya[4] += c5 + b[4] * t5;
  yb[4] += c5 - a[4] * t5;
  const double f4 = F1 * m4;
  const double s1 = 0.5 * (F1 * m1 + m4 * p_hat + A * rho_ln) + f4 * u, s2 = 0.5 * F1 * m2 + f4 * v,
               s3 = 0.5 * F1 * m3 + f4 * w;
  ya[1] += s1 - f4 * a[1];
  yb[1] += s1 - f4 * b[1];
  ya[2] += s2 - f4 * a[2];
  yb[2] += s2 - f4 * b[2];
  ya[3] += s3 - f4 * a[3];
  yb[3] += s3 - f4 * b[3];
}

// All pairs of a line.  A line of eight nodes with its cotangents and sums exceeds the
// registers: blocks of four, the second block's nodes one by one against the first.
template <int N, bool EC>
__device__ __forceinline__ void line_pairs(const DevBasis& b, const double* sF, const LineTask<N>& t, double c, double kap,
                                           double (&y)[N + 1][6]) {
  constexpr int NP = N + 1, H = VjpShape<N>::BLOCK;
  double x[H][11];
  const auto pair = [&](const double (&p)[11], const double (&q)[11], int i, int m) {
    if constexpr (EC)
      ec_pair_vjp<0>(p, q, q_im<N, double>(b, i, m), kap, y[i], y[m]);
    else
      kg_pair_vjp(p, q, q_im<N, double>(b, i, m), y[i], y[m]);
  };
#pragma unroll
  for (int b0 = 0; b0 < NP; b0 += H) {
#pragma unroll
    for (int i = 0; i < H; ++i) vjp_node<N, EC>(sF, b.inv_w, t, b0 + i, c, x[i]);
    if (EC) settle(x);  // (nothing of the versions is shared, and held, before the branch)
#pragma unroll
    for (int i = 0; i < H; ++i)
#pragma unroll
      for (int m = i + 1; m < H; ++m) {
        pair(x[i], x[m], b0 + i, b0 + m);
        if (EC || m % 2) __builtin_amdgcn_sched_barrier(0);
      }
    if (b0 == 0)
#pragma unroll
      for (int m = H; m < NP; ++m) {
        double z[11];
        vjp_node<N, EC>(sF, b.inv_w, t, m, c, z);
#pragma unroll
        for (int i = 0; i < H; ++i) {
          pair(x[i], z, i, m);
          if (EC || i % 2) __builtin_amdgcn_sched_barrier(0);
        }
      }
  }
}

// The same with larger jumps (MEANS 1 or 2), not unrolled (further unrolled versions
// spill registers into the usual one): the sums of row m are selected by factors 0 and 1.
template <int N, int MEANS>
__device__ inline void line_rows_ec(const DevBasis& b, const double* sF, const double* sW, const LineTask<N>& t, double c,
                                    double kap, double (&y)[N + 1][6]) {
  constexpr int NP = N + 1;
#pragma unroll 1
  for (int i = 0; i < N; ++i) {
    double x[11], z[6] = {0, 0, 0, 0, 0, 0};
    vjp_node<N, true>(sF, sW, t, i, c, x);
#pragma unroll 1
    for (int m = i + 1; m < NP; ++m) {
      double q[11], f[6] = {0, 0, 0, 0, 0, 0};
      vjp_node<N, true>(sF, sW, t, m, c, q);
      ec_pair_vjp<MEANS>(x, q, q_im<N, double>(b, i, m), kap, z, f);
#pragma unroll
      for (int r = 1; r < NP; ++r) {
        const double sel = r == m ? 1.0 : 0.0;
#pragma unroll
        for (int v = 0; v < 5; ++v) y[r][v] += sel * f[v];
      }
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const double sel = r == i ? 1.0 : 0.0;
#pragma unroll
      for (int v = 0; v < 5; ++v) y[r][v] += sel * z[v];
    }
  }
}

// Cotangent of the own state Ub, line frame, through one face's convective flux F*: P own
// primitives (rho, u, v, w, p, e), lo own lam, sn and ln of the neighbour,
// so_iw and sn_iw the two elements' s_d / w_end.  The own side is L of an upper face.
// (In the weak form the own physical flux cancels with the diagonal of the volume sum.)
// The dissipation's cotangent belongs to the conservative state: through those of (rho, e)
// it would cancel again in rho, behind the rounding of e times the wave speed.
template <bool EC>
__device__ __forceinline__ void face_vjp(const DevPhys& ph, const double (&P)[6], const double (&lo)[5],
                                         const double (&sn)[5], const double (&ln)[5], bool wall, bool up, double so_iw,
                                         double sn_iw, double (&Ub)[5]) {
  double Pb[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int v = 0; v < 5; ++v) Ub[v] = 0.0;
  const double sg = up ? -1.0 : 1.0;
  if (wall) {  // F*_c = (0, p_o e_d, 0)
    Pb[4] = sg * so_iw * lo[1];
    prim_vjp(P, Pb, 0.0, ph, Ub);
    return;
  }
  double phi[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) phi[v] = sg * (so_iw * lo[v] - sn_iw * ln[v]);
  double Pn[6];
  to_prim(sn, ph, Pn);
  const double so[5] = {P[0], P[0] * P[1], P[0] * P[2], P[0] * P[3], P[0] * P[5]};
  if constexpr (EC) {
    // F*_c = f#_EC(U_L, U_R) - (1/2) Roe(U_L, U_R)
    const double Ae[6] = {P[0], P[1], P[2], P[3], P[4], 0.5 * P[0] / P[4]};
    const double Be[6] = {Pn[0], Pn[1], Pn[2], Pn[3], Pn[4], 0.5 * Pn[0] / Pn[4]};
    double Pbe[6] = {0, 0, 0, 0, 0, 0};
    ec_vjp(Ae, Be, phi, ph.gm1, Pbe);
    fold_beta(Ae, Pbe, Pb);
    if (!ph.central) roe_vjp(so, sn, up, phi, ph, Pb);
  } else {
    kg_vjp(P, Pn, phi, Pb);
    if (!ph.central) {
      const double co = fabs(P[1]) + sqrt(ph.gamma * P[4] / P[0]);
      const double cn = fabs(Pn[1]) + sqrt(ph.gamma * Pn[4] / Pn[0]);
      const double lam = up ? (co >= cn ? co : cn) : (cn >= co ? cn : co);
      const bool own_active = up ? (co >= cn) : (co > cn);
      // F*_c contains -lam/2 (U_R - U_L)
      const double dU = up ? 0.5 * lam : -0.5 * lam;
      double lb = 0.0;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        Ub[v] = dU * phi[v];
        lb -= 0.5 * phi[v] * (up ? sn[v] - so[v] : so[v] - sn[v]);
      }
      if (own_active) speed_vjp(P, lb, ph, Pb);
    }
  }
  prim_vjp(P, Pb, 0.0, ph, Ub);
}

// ROLE 0: line lanes, 1: face lanes, 2: neither (the node phases only).
template <int N, bool EC, int ROLE>
__device__ __forceinline__ void vjp_phases(const VjpArgsPtr args, double* const head, const int e, const int tid) {
  using L = Line<N>;
  using S = VjpShape<N>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, LINES = L::LINES;
  double* const sW = head;
  double* const sF = head + S::HEAD;
  double y[NP][6];     // line lanes: cotangents of the line's nodes
  double ue[2][5];     // face lanes: those of the states at its ends, through the faces
  const Place pl(again(args).mesh, e);
  const bool visc = again(args).ph.viscous != 0;
  {
    const VjpArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
    const unsigned n = tid < NN ? tid : 0;
    double u[5], l[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = (A.U + v * stride + static_cast<long long>(e) * NN)[n];
#pragma unroll
    for (int v = 0; v < 5; ++v) l[v] = (A.lam + v * stride + static_cast<long long>(e) * NN)[n];
    if (tid < NP) {
      double w = A.basis.inv_w[0];
#pragma unroll
      for (int i = 1; i < NP; ++i) w = tid == i ? A.basis.inv_w[i] : w;
      sW[tid] = w;
    }
    double sn[2][5], ln[2][5], s_n[2];  // the neighbours' at the line's ends
    if constexpr (ROLE == 1) {
      const LineTask<N> t(tid - 64 * S::LW);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        fetch_end<N>(A.U, stride, pl, e, t, h, sn[h]);
        fetch_end<N>(A.lam, stride, pl, e, t, h, ln[h]);
        s_n[h] = nb_scale(A.mesh, pl.ex, pl.ey, pl.ez, t.d, h != 0);
      }
    }
    if (tid < NN) {
      double P[6];
      to_prim(u, A.ph, P);
      const int p = L::at(n % NP, (n / NP) % NP, n / NF);
#pragma unroll
      for (int q = 0; q < 4; ++q) sF[q * EB + p] = 0.5 * P[q];
      if (EC) {
        sF[4 * EB + p] = 0.5 * P[0] / P[4];
      } else {
        sF[4 * EB + p] = 0.5 * P[4];
        sF[5 * EB + p] = 0.5 * P[5];
      }
      sF[S::T * EB + p] = P[4] * A.ph.inv_R / P[0];
#pragma unroll
      for (int v = 0; v < 5; ++v) sF[(S::LAM + v) * EB + p] = l[v];
    }
    phase_end();

    // ---- pairs on the line waves; faces and derivatives on the face waves ----
    if constexpr (ROLE == 1) {
      const VjpArgs& B = again(args);
      const LineTask<N> t(again(tid) - 64 * S::LW);
      const double iw = B.basis.inv_w[0];
      const double s = t.d == 0 ? pl.sx : (t.d == 1 ? pl.sy : pl.sz);
      double gl[2][4], gq[2][4];  // ghosts: lam (momentum, energy) s / w; u, v, w (halves), T
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int p = t.node(h ? N : 0);
        const bool wall = pl.neighbour(t.d, h) < 0;
        const double siw = s * iw, niw = iw * s_n[h];
        const double r = 2.0 * sF[p], T = sF[S::T * EB + p];
        double P[6] = {r, 2.0 * sF[(1 + t.d) * EB + p], 2.0 * sF[(1 + t.d1) * EB + p], 2.0 * sF[(1 + t.d2) * EB + p], 0, 0};
        if (EC) {
          P[4] = 0.5 * r / sF[4 * EB + p];
          P[5] = P[4] / (B.ph.gm1 * r) + 0.5 * (P[1] * P[1] + P[2] * P[2] + P[3] * P[3]);
        } else {
          P[4] = 2.0 * sF[4 * EB + p];
          P[5] = 2.0 * sF[5 * EB + p];
        }
        const double lo[5] = {sF[S::LAM * EB + p], sF[(S::LAM + 1 + t.d) * EB + p], sF[(S::LAM + 1 + t.d1) * EB + p],
                              sF[(S::LAM + 1 + t.d2) * EB + p], sF[(S::LAM + 4) * EB + p]};
        face_vjp<EC>(B.ph, P, lo, sn[h], ln[h], wall, h != 0, siw, niw, ue[h]);
        const double ir = rcp_nr(sn[h][0]);
        const double v0 = sn[h][1] * ir, v1 = sn[h][2] * ir, v2 = sn[h][3] * ir;
        const double Tn = B.ph.gm1 * (sn[h][4] - 0.5 * (sn[h][1] * v0 + sn[h][2] * v1 + sn[h][3] * v2)) * B.ph.inv_R * ir;
#pragma unroll
        for (int c = 0; c < 4; ++c) gl[h][c] = wall ? siw * lo[1 + c] : -niw * ln[h][1 + c];
        gq[h][0] = wall ? -0.5 * P[1] : 0.5 * v0;
        gq[h][1] = wall ? -0.5 * P[2] : 0.5 * v1;
        gq[h][2] = wall ? -0.5 * P[3] : 0.5 * v2;
        gq[h][3] = wall ? 2.0 * B.mesh.T_wall - T : Tn;
      }
      settle(ue);
      settle(gl);
      settle(gq);
      if (visc) {
        // lam of momentum and energy -> the flux cotangents -w s dlam/dx (a wall's flux
        // takes the own stresses and heat flux: ghost -lam); u, v, w, T -> gradients
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int v = c & 3, k = v == 0 ? t.d : (v == 1 ? t.d1 : (v == 2 ? t.d2 : 3));
          const int src = c < 4 ? S::LAM + 1 + k : (v == 3 ? S::T : 1 + k);
          double q[NP], g[NP];
#pragma unroll
          for (int m = 0; m < NP; ++m) q[m] = sF[src * EB + t.node(m)];
          if (c < 4)
#pragma unroll
            for (int m = 0; m < NP; ++m) q[m] *= -s * B.basis.inv_w[m];
          line_derivative<N, double, false>(B.basis, q, c < 4 ? gl[0][v] : gq[0][v], c < 4 ? gl[1][v] : gq[1][v], g);
#pragma unroll
          for (int m = 0; m < NP; ++m) sF[((c < 4 ? S::FV : S::GR) + 3 * k + t.d) * EB + t.node(m)] = g[m];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  if constexpr (ROLE == 0) {
    const VjpArgs& A = again(args);
    const LineTask<N> t(again(tid));
    const double s = t.d == 0 ? pl.sx : (t.d == 1 ? pl.sy : pl.sz);
#pragma unroll
    for (int m = 0; m < NP; ++m)
#pragma unroll
      for (int v = 0; v < 6; ++v) y[m][v] = 0.0;
    if constexpr (EC) {
      // f of the largest pair is that of the line's extremes: small for rho and beta
      // on all lines of the wave, all means take their series
      double lo[2], hi[2];
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        const double r = sF[t.node(m)], be = sF[4 * EB + t.node(m)];
        lo[0] = m == 0 || r < lo[0] ? r : lo[0];
        hi[0] = m == 0 || r > hi[0] ? r : hi[0];
        lo[1] = m == 0 || be < lo[1] ? be : lo[1];
        hi[1] = m == 0 || be > hi[1] ? be : hi[1];
      }
      const double dr = hi[0] - lo[0], sr = hi[0] + lo[0], db = hi[1] - lo[1], sb = hi[1] + lo[1];
      const bool mid = dr >= 0.01 * sr || db >= 0.01 * sb, large = dr >= 0.1 * sr || db >= 0.1 * sb;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(large) != 0, 0))
        line_rows_ec<N, 2>(A.basis, sF, sW, t, -2.0 * s, 0.5 / A.ph.gm1, y);
      else if (__builtin_amdgcn_ballot_w64(mid) != 0)
        line_rows_ec<N, 1>(A.basis, sF, sW, t, -2.0 * s, 0.5 / A.ph.gm1, y);
      else
        line_pairs<N, true>(A.basis, sF, t, -2.0 * s, 0.5 / A.ph.gm1, y);
    } else {
      line_pairs<N, false>(A.basis, sF, t, -s, 0.0, y);
    }
    settle(y);
  }
  phase_end();

  // ---- node phase: transposed viscous flux ----------------------------------
  double Pu[3] = {0, 0, 0}, Tb = 0.0;
  const int tn = again(tid);
  const unsigned n = tn < NN ? tn : 0;
  const int i = n % NP, j = (n / NP) % NP, k = n / NF, l = L::at(i, j, k);
  if (visc && tn < NN) {
    const VjpArgs& A = again(args);
    const double c[3] = {2.0 * (pl.sx * sW[i]), 2.0 * (pl.sy * sW[j]), 2.0 * (pl.sz * sW[k])};
    const double T = sF[S::T * EB + l], rT = viscosity_ratio(A.ph, T);
    const double mu = A.ph.mu * rT, kappa = A.ph.kappa * rT;
    double g[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) g[q] = c[q % 3] * sF[(S::GR + q) * EB + l];
    const double l4 = 0.5 * sF[(S::LAM + 4) * EB + l];
    double tb[9], gT[3], eb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int x = d == 0 ? i : (d == 1 ? j : k);
      gT[d] = sF[(S::FV + 9 + d) * EB + l];
      // a wall's energy flux is without the stresses' work
      const double om = (x == 0 && pl.nb[2 * d] < 0 ? c[d] * l4 : 0.0) - (x == N && pl.nb[2 * d + 1] < 0 ? c[d] * l4 : 0.0);
      eb[d] = gT[d] + om;
#pragma unroll
      for (int q = 0; q < 3; ++q) tb[3 * q + d] = sF[(S::FV + 3 * q + d) * EB + l] + eb[d] * (2.0 * sF[(1 + q) * EB + l]);
    }
    const double dv = (2.0 / 3.0) * (g[0] + g[4] + g[8]), tr = (2.0 / 3.0) * mu * (tb[0] + tb[4] + tb[8]);
    const long long stride = A.mesh.nE * NN;
    double* out = A.gbar + static_cast<long long>(e) * NN;
    double st = 0.0;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int y2 = 0; y2 < 3; ++y2) {
        const double gb = mu * (tb[3 * x + y2] + tb[3 * y2 + x]) - (x == y2 ? tr : 0.0);
        store_once(&(out + (3 * x + y2) * stride)[n], gb);
        st += gb * g[3 * x + y2];
        Pu[x] += eb[y2] * (mu * (g[3 * x + y2] + g[3 * y2 + x] - (x == y2 ? dv : 0.0)));
      }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      store_once(&(out + (9 + d) * stride)[n], kappa * gT[d]);
      st += kappa * gT[d] * (0.5 * c[d] * sF[(S::GR + 9 + d) * EB + l]);
    }
    // Sutherland's law: tau and q scale with r(T), d ln r / dT = 3 / (2 T) - 1 / (T + S)
    if (A.ph.suth) Tb = (1.5 / T - 1.0 / (T + A.ph.suth_S)) * st;
  }
  phase_end();

  // ---- sums of the lines and faces, transposed primitive map ----------------
  if constexpr (ROLE == 0) {
    const LineTask<N> t(again(tid));
    double* o = sF + (S::SUM + 6 * t.d) * EB;
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int p = t.node(m);
      o[p] = y[m][0];
      o[(1 + t.d) * EB + p] = y[m][1];
      o[(1 + t.d1) * EB + p] = y[m][2];
      o[(1 + t.d2) * EB + p] = y[m][3];
      o[4 * EB + p] = y[m][4];
      if (!EC) o[5 * EB + p] = y[m][5];
    }
  } else if constexpr (ROLE == 1) {
    const LineTask<N> t(again(tid) - 64 * S::LW);
    double* o = sF + S::END + t.d * NF + t.ab;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      o[(5 * h) * LINES] = ue[h][0];
      o[(5 * h + 1 + t.d) * LINES] = ue[h][1];
      o[(5 * h + 1 + t.d1) * LINES] = ue[h][2];
      o[(5 * h + 1 + t.d2) * LINES] = ue[h][3];
      o[(5 * h + 4) * LINES] = ue[h][4];
    }
  }
  phase_end();
  if (tn < NN) {
    const VjpArgs& A = again(args);
    double Pb[6] = {0, Pu[0], Pu[1], Pu[2], 0, 0};
#pragma unroll
    for (int q = 0; q < (EC ? 5 : 6); ++q)
#pragma unroll
      for (int d = 0; d < 3; ++d) Pb[q] += sF[(S::SUM + 6 * d + q) * EB + l];
    double P[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) P[q] = EC && q > 3 ? 0.0 : 2.0 * sF[q * EB + l];
    if (EC) {
      const double beta = sF[4 * EB + l];
      P[4] = 0.5 * P[0] / beta;
      P[5] = P[4] / (A.ph.gm1 * P[0]) + 0.5 * (P[1] * P[1] + P[2] * P[2] + P[3] * P[3]);
      const double Ae[6] = {P[0], 0, 0, 0, P[4], beta}, Pbe[6] = {0, 0, 0, 0, 0, Pb[4]};
      Pb[4] = 0.0;
      fold_beta(Ae, Pbe, Pb);
    }
    double Ub[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int x = d == 0 ? i : (d == 1 ? j : k);
      if (x == 0 || x == N) {
        const int ab = d == 0 ? j + NP * k : (d == 1 ? i + NP * k : i + NP * j);
        const double* o = sF + S::END + (x == N ? 5 : 0) * LINES + d * NF + ab;
#pragma unroll
        for (int v = 0; v < 5; ++v) Ub[v] += o[v * LINES];
      }
    }
    prim_vjp(P, Pb, Tb, A.ph, Ub);
    const long long stride = A.mesh.nE * NN;
#pragma unroll
    for (int v = 0; v < 5; ++v) store_once(&(A.ubar + v * stride + static_cast<long long>(e) * NN)[n], Ub[v]);
  }
}

template <int N, bool EC>
__global__ __launch_bounds__(VjpShape<N>::BS) __attribute__((amdgpu_waves_per_eu(2))) void k_vjp_a(VjpArgs) {
  extern __shared__ double lds[];
  const VjpArgsPtr args = (VjpArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid) / 64;
  const int e = xcd_remap(blockIdx.x, gridDim.x);
  constexpr int LW = VjpShape<N>::LW;
  if (wave < LW)
    vjp_phases<N, EC, 0>(args, lds, e, tid);
  else if (2 * LW * 64 == VjpShape<N>::BS || wave < 2 * LW)
    vjp_phases<N, EC, 1>(args, lds, e, tid);
  else
    vjp_phases<N, EC, 2>(args, lds, e, tid);
}

// --------------------------------------------------------------------------
// k_vjp_b: transposed lifting
// --------------------------------------------------------------------------
template <int N, bool ACC>
__global__ __launch_bounds__(Cfg<N>::BS) void k_vjp_b(const double* __restrict__ U,
                                                       const double* __restrict__ gbar,
                                                       const double* __restrict__ ubar,
                                                       double* __restrict__ out, double scale,
                                                       double* __restrict__ cot, double cot_a,
                                                       double cot_b, DevMesh mesh, DevPhys ph,
                                                       DevBasis basis) {
  using Gm = Geo<N>;
  constexpr int NP = Gm::NP, NF = Gm::NF, NN = Gm::NN, EB = Gm::EB, DS = Gm::DS;
  constexpr int EPB = Cfg<N>::EPB, BS = Cfg<N>::BS;
  __shared__ double sD[NP * DS];
  __shared__ double sG[EPB][12][EB];
  __shared__ double sQ[EPB][6][4][NF];

  const int tid = threadIdx.x;
  const long long nE = mesh.nE;
  const long long stride = nE * NN;
  const long long e0 = static_cast<long long>(xcd_remap(blockIdx.x, gridDim.x)) * EPB;
  for (int t = tid; t < NP * NP; t += BS) sD[(t / NP) * DS + t % NP] = basis.D[t];
  int ex0 = 0, ey0 = 0, ez0 = 0;
  elem_coords(e0 < nE ? e0 : 0, mesh, ex0, ey0, ez0);

  const int le = EPB == 1 ? 0 : tid / NN;
  const int node = tid - le * NN;
  const long long e = EPB == 1 ? e0 : e0 + le;
  const bool active = (EPB == 1 ? tid < NN : le < EPB) && e < nE;
  const int i = node % NP, j = (node / NP) % NP, k = node / NF;
  const int l = Gm::lds(i, j, k);
  const bool visc = ph.viscous != 0;

  if (active && visc) {
#pragma unroll
    for (int c = 0; c < 12; ++c) sG[le][c][l] = gbar[c * stride + e * NN + node];
  }
  __syncthreads();
  if (visc && tid < n_face_tasks<N>()) {
    const FaceTask<N> ft(tid);
    const long long te = EPB == 1 ? e0 : e0 + ft.le;
    if (te < nE) {
      int fx = ex0, fy = ey0, fz = ez0;
      if (EPB > 1) elem_coords(te, mesh, fx, fy, fz);
      const long long nb = neighbour(mesh, fx, fy, fz, ft.d, ft.up);
      const double s_o = mesh.s[ft.d][ft.d == 0 ? fx : (ft.d == 1 ? fy : fz)];
      const double sgn = (ft.up ? -1.0 : 1.0) * basis.inv_w_end;
      const int lo = Gm::lds(ft.oi, ft.oj, ft.ok);
      if (nb < 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) sQ[ft.le][ft.f][c][ft.ab] = sgn * s_o * sG[ft.le][3 * c + ft.d][lo];
      } else {
        const double s_n = nb_scale(mesh, fx, fy, fz, ft.d, ft.up);
        const long long nidx = nb * NN + ft.nb_node();
#pragma unroll
        for (int c = 0; c < 4; ++c)
          sQ[ft.le][ft.f][c][ft.ab] =
              0.5 * sgn * (s_o * sG[ft.le][3 * c + ft.d][lo] + s_n * gbar[(3 * c + ft.d) * stride + nidx]);
      }
    }
  }
  __syncthreads();
  if (!active) return;

  int ex = ex0, ey = ey0, ez = ez0;
  if (EPB > 1) elem_coords(e, mesh, ex, ey, ez);
  const long long idx = e * NN + node;
  double Ub[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) Ub[v] = load_once(&ubar[v * stride + idx]);
  if (visc) {
    const double sx = mesh.s[0][ex], sy = mesh.s[1][ey], sz = mesh.s[2][ez];
    double qb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double ax = 0.0, ay = 0.0, az = 0.0;
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        ax += sD[m * DS + i] * sG[le][3 * c + 0][Gm::lds(m, j, k)];
        ay += sD[m * DS + j] * sG[le][3 * c + 1][Gm::lds(i, m, k)];
        az += sD[m * DS + k] * sG[le][3 * c + 2][Gm::lds(i, j, m)];
      }
      qb[c] = sx * ax + sy * ay + sz * az;
      if (i == 0) qb[c] += sQ[le][0][c][j + NP * k];
      if (i == N) qb[c] += sQ[le][1][c][j + NP * k];
      if (j == 0) qb[c] += sQ[le][2][c][i + NP * k];
      if (j == N) qb[c] += sQ[le][3][c][i + NP * k];
      if (k == 0) qb[c] += sQ[le][4][c][i + NP * j];
      if (k == N) qb[c] += sQ[le][5][c][i + NP * j];
    }
    double s[5], P[6];
    load_state(U, stride, idx, s);
    to_prim(s, ph, P);
    const double Pb[6] = {0.0, qb[0], qb[1], qb[2], 0.0, 0.0};
    prim_vjp(P, Pb, qb[3], ph, Ub);
  }
  if (ACC) {
    // out += scale Ubar; with cot, also the next RK stage cotangent
    // cot <- cot_a cot + cot_b out at this node (no workgroup reads cot here)
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double nv = load_once(&out[v * stride + idx]) + scale * Ub[v];
      store_once(&out[v * stride + idx], nv);
      if (cot) store_once(&cot[v * stride + idx], cot_a * load_once(&cot[v * stride + idx]) + cot_b * nv);
    }
  } else {
#pragma unroll
    for (int v = 0; v < 5; ++v) store_once(&out[v * stride + idx], Ub[v]);
  }
}

// y = a y + b x; with a = 0 the old y is not read (a cleared or never written
// buffer may hold anything), with x null y = a y.
__global__ void k_axpby(double* __restrict__ y, const double* __restrict__ x, double a, double b,
                        long long n) {
  for (long long t = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x; t < n;
       t += static_cast<long long>(gridDim.x) * blockDim.x) {
    const double ay = a == 0.0 ? 0.0 : a * load_once(&y[t]);
    store_once(&y[t], x ? ay + b * load_once(&x[t]) : ay);
  }
}

template <int N>
hipError_t vjp_n(const DevMesh& m, const DevPhys& p, const DevBasis& b, const double* U,
                 const double* lam, double* gbar, double* ubar, double* out,
                 bool acc, double scale, double* cot, double cot_a, double cot_b, hipStream_t s) {
  const VjpArgs a{U, lam, gbar, ubar, m, p, b};
  const dim3 grid(static_cast<unsigned>(m.nE)), block(VjpShape<N>::BS);
  if (p.ec)
    hipLaunchKernelGGL((k_vjp_a<N, true>), grid, block, VjpShape<N>::BYTES, s, a);
  else
    hipLaunchKernelGGL((k_vjp_a<N, false>), grid, block, VjpShape<N>::BYTES, s, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (acc)
    hipLaunchKernelGGL((k_vjp_b<N, true>), dim3(n_blocks<N>(m.nE)), dim3(Cfg<N>::BS), 0, s, U,
                       gbar, ubar, out, scale, cot, cot_a, cot_b, m, p, b);
  else
    hipLaunchKernelGGL((k_vjp_b<N, false>), dim3(n_blocks<N>(m.nE)), dim3(Cfg<N>::BS), 0, s, U,
                       gbar, ubar, out, scale, static_cast<double*>(nullptr), 0.0, 0.0, m, p, b);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rhs_vjp(int N, const DevMesh& m, const DevPhys& p, const DevBasis& b,
                          const double* U, const double* lam, double* gbar, double* ubar,
                          double* out, bool accumulate, double scale, hipStream_t s, double* cot,
                          double cot_a, double cot_b) {
  if (m.nE <= 0) return hipSuccess;
  if (cot && !accumulate) return hipErrorInvalidValue;
  switch (N) {
    case 3: return vjp_n<3>(m, p, b, U, lam, gbar, ubar, out, accumulate, scale, cot, cot_a, cot_b, s);
    case 5: return vjp_n<5>(m, p, b, U, lam, gbar, ubar, out, accumulate, scale, cot, cot_a, cot_b, s);
    case 7: return vjp_n<7>(m, p, b, U, lam, gbar, ubar, out, accumulate, scale, cot, cot_a, cot_b, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_axpby(double* y, const double* x, double a, double b, long long n, hipStream_t s) {
  long long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_axpby, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, y, x, a, b, n);
  return hipGetLastError();
}

}  // namespace dg
