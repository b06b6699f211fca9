// Split-form DGSEM on curvilinear hexahedra (FP64 or mixed precision,
// structured meshes with periodic or isothermal no-slip wall ends).
//
// Geometry (the paper's production meshes are curved, Sec. 4): each element's
// map is the degree-N interpolant of its node coordinates.  The metric terms
// J a^i_n are Kopriva's conservative curl form,
//   J a^i_n = -1/2 [curl_xi (X_l grad_xi X_m - X_m grad_xi X_l)]_i, (n, m, l) cyclic,
// with the collocation derivative D for every xi-derivative, so the discrete
// metric identities hold and both elements of a face see the same normal;
// J = det(dX/dxi).  k_metrics computes them once per mesh into
//   geo[c][e][node], c = 3 i + n: J a^i_n; c = 9: 1 / J; then the same ten
//   fields in FP32 (read by the mixed-precision sweeps).
// Operator per stage (one workgroup per element, one lane per node; face
// lanes = one lane per face node):
//   k_face_flux_curv  BR1 gradients at the face nodes (chain rule with the
//                     node's metrics: J grad q = sum_i J a^i (D_i q + lifting
//                     term)) and the contravariant normal viscous flux
//                     Fv^i = sum_d f_v,d J a^i_d of every face, to ffv;
//   k_rhs_curv        gradients of every node, per direction i the
//                     contravariant Kennedy-Gruber two-point flux with
//                     averaged metrics sum_d f#_d (J a^i_d(A) + J a^i_d(B)) / 2
//                     and the viscous flux Fv^i, Lax-Friedrichs across each
//                     face with its normal J a^i (that of the element below
//                     the face, shared by both sides), Ut = -(1/J)(...),
//                     fused RK update.
#include "curv_flux.hpp"

namespace dg {
namespace {

template <int N>
struct CurvCfg {
  static constexpr int NP = N + 1, NF = NP * NP, NN = NF * NP;
  static constexpr int LANES = NN > 6 * NF ? NN : 6 * NF;
  static constexpr int BS = (LANES + 63) / 64 * 64;
};

// sum_m D[idx][m] f(node with the dir-coordinate replaced by m), f an LDS field
// indexed i + NP (j + NP k)
template <int N, typename R>
__device__ inline R dline(const R* f, const double (*sD)[N + 2], int dir, int i, int j, int k) {
  constexpr int NP = N + 1;
  const int idx = dir == 0 ? i : (dir == 1 ? j : k);
  const int base = dir == 0 ? NP * (j + NP * k) : (dir == 1 ? i + NP * NP * k : i + NP * j);
  const int step = dir == 0 ? 1 : (dir == 1 ? NP : NP * NP);
  R a = R(0);
#pragma unroll
  for (int m = 0; m < NP; ++m) a += static_cast<R>(sD[idx][m]) * f[base + step * m];
  return a;
}

// ---------------------------------------------------------------- metrics
template <int N>
__global__ __launch_bounds__(CurvCfg<N>::BS) void k_metrics(const double* __restrict__ X,
                                                           double* __restrict__ geo,
                                                           double* __restrict__ geoF, bool with_f32,
                                                           DevBasis basis, long long nE,
                                                           int* __restrict__ status) {
  using C = CurvCfg<N>;
  constexpr int NP = C::NP, NN = C::NN;
  __shared__ double sD[NP][N + 2];
  __shared__ double sX[3][NN];
  __shared__ double sdX[9][NN];  // dX_n / dxi^j at 3 n + j
  __shared__ double sV[3][NN];
  const int tid = threadIdx.x;
  const long long e = blockIdx.x;
  const long long stride = nE * NN;
  const bool active = tid < NN;
  const int i = tid % NP, j = (tid / NP) % NP, k = tid / (NP * NP);
  if (tid < NP * NP) sD[tid / NP][tid % NP] = basis.D[tid];
  // coordinates relative to the element's node (0, 0, 0): the curl form is
  // translation invariant, and its rounding then scales with the element's
  // size instead of the magnitude of the coordinates
  if (active) {
#pragma unroll
    for (int n = 0; n < 3; ++n) sX[n][tid] = X[n * stride + e * NN + tid] - X[n * stride + e * NN];
  }
  __syncthreads();
  double dX[9];
  if (active) {
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        dX[3 * n + d] = dline<N>(sX[n], sD, d, i, j, k);
        sdX[3 * n + d][tid] = dX[3 * n + d];
      }
  }
  __syncthreads();
  double Ja[9];
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    const int m = (n + 1) % 3, l = (n + 2) % 3;
    if (active) {
#pragma unroll
      for (int d = 0; d < 3; ++d)
        sV[d][tid] = sX[l][tid] * sdX[3 * m + d][tid] - sX[m][tid] * sdX[3 * l + d][tid];
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int a = (r + 1) % 3, b = (r + 2) % 3;
        Ja[3 * r + n] = -0.5 * (dline<N>(sV[b], sD, a, i, j, k) - dline<N>(sV[a], sD, b, i, j, k));
      }
    }
    __syncthreads();
  }
  if (active) {
    const double J = dX[0] * (dX[4] * dX[8] - dX[5] * dX[7]) - dX[1] * (dX[3] * dX[8] - dX[5] * dX[6]) +
                     dX[2] * (dX[3] * dX[7] - dX[4] * dX[6]);
    if (!(J > 0.0)) status[0] = 1;
    const long long o = e * NN + tid;
#pragma unroll
    for (int c = 0; c < 9; ++c) geo[c * stride + o] = Ja[c];
    geo[9 * stride + o] = 1.0 / J;
    // boundary nodes once more, contiguous per element (face node number t)
    if (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N) {
      constexpr int NFN = n_face_nodes<N>();
      const long long of = e * NFN + face_node_index<N>(i, j, k);
#pragma unroll
      for (int c = 0; c < 9; ++c) geoF[c * nE * NFN + of] = Ja[c];
      geoF[9 * nE * NFN + of] = 1.0 / J;
    }
    // FP32 copy for the mixed-precision sweeps, after the ten FP64 fields
    // (the workspace holds it only in mixed-precision contexts)
    if (with_f32) {
      float* const g32 = reinterpret_cast<float*>(geo + 10 * stride);
#pragma unroll
      for (int c = 0; c < 9; ++c) g32[c * stride + o] = static_cast<float>(Ja[c]);
      g32[9 * stride + o] = static_cast<float>(1.0 / J);
    }
  }
}

// Physical gradients of q = (u, v, w, T) at node (i, j, k): reference
// derivatives plus the lifting terms of the faces the node lies on, then
// grad q = (1/J) sum_r J a^r gxi_r.  sq[c] are LDS fields of q; corr[f][c][ab]
// the lifting terms (q* - q)(+-1/w) of face f.
template <int N, typename R>
__device__ inline void curv_gradients(const R* const sq[4], const double (*sD)[N + 2],
                                      const R (*corr)[4][(N + 1) * (N + 1)], int i, int j, int k,
                                      const R Ja[9], R invJ, R g[12]) {
  constexpr int NP = N + 1;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    R gx[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) gx[r] = dline<N, R>(sq[c], sD, r, i, j, k);
    if (i == 0) gx[0] += corr[0][c][j + NP * k];
    if (i == N) gx[0] += corr[1][c][j + NP * k];
    if (j == 0) gx[1] += corr[2][c][i + NP * k];
    if (j == N) gx[1] += corr[3][c][i + NP * k];
    if (k == 0) gx[2] += corr[4][c][i + NP * j];
    if (k == N) gx[2] += corr[5][c][i + NP * j];
#pragma unroll
    for (int d = 0; d < 3; ++d) g[3 * c + d] = invJ * (Ja[d] * gx[0] + Ja[3 + d] * gx[1] + Ja[6 + d] * gx[2]);
  }
}

// ---------------------------------------------------------- face viscous flux
// (R = float in mixed precision: the fluxes are formed in FP64 and stored in FP32)
template <int N, typename R>
__global__ __launch_bounds__(CurvCfg<N>::BS) void k_face_flux_curv(const double* __restrict__ U,
                                                                  R* __restrict__ ffv, DevMesh mesh,
                                                                  DevPhys ph, DevBasis basis) {
  using C = CurvCfg<N>;
  constexpr int NP = C::NP, NF = C::NF, NN = C::NN;
  __shared__ double sD[NP][N + 2];
  __shared__ double sq[4][NN];
  __shared__ double corr[6][4][NF];
  const int tid = threadIdx.x;
  const long long nE = mesh.nE;
  const long long stride = nE * NN;
  const long long e = xcd_remap(blockIdx.x, gridDim.x);
  int ex, ey, ez;
  elem_coords(e, mesh, ex, ey, ez);
  if (tid < NP * NP) sD[tid / NP][tid % NP] = basis.D[tid];
  constexpr int NFN = n_face_nodes<N>();
  static_assert(NFN <= CurvCfg<N>::BS, "one lane per boundary node");
  double Ja[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, invJ = 0.0;
  if (tid < NFN) {
    const long long fs = nE * NFN, of = e * NFN + tid;
#pragma unroll
    for (int c = 0; c < 9; ++c) Ja[c] = mesh.geoF[c * fs + of];
    invJ = mesh.geoF[9 * fs + of];
  }
  if (tid < NN) {
    double s[5];
    load_state(U, stride, e * NN + tid, s);
    const Prim P = primitives(s, ph);
    sq[0][tid] = P.u;
    sq[1][tid] = P.v;
    sq[2][tid] = P.w;
    sq[3][tid] = P.T;
  }
  // face lanes fetch the neighbour's face node now and take their own values
  // from LDS after the barrier
  double sn[5] = {1.0, 0.0, 0.0, 0.0, 1.0};
  long long nb = -1;  // -1: the face is a wall
  if (tid < 6 * NF) {
    const FaceTask<N> ft(tid);
    nb = neighbour(mesh, ex, ey, ez, ft.d, ft.up);
    if (nb >= 0) load_state(U, stride, nb * NN + ft.nb_node(), sn);
  }
  __syncthreads();
  if (tid < 6 * NF) {
    const FaceTask<N> ft(tid);
    const int lo = ft.own_node();
    const double qo[4] = {sq[0][lo], sq[1][lo], sq[2][lo], sq[3][lo]};
    double qs[4] = {0.0, 0.0, 0.0, mesh.T_wall};  // isothermal no-slip wall
    if (nb >= 0) {
      const Prim Pn = primitives(sn, ph);
      qs[0] = 0.5 * (qo[0] + Pn.u);
      qs[1] = 0.5 * (qo[1] + Pn.v);
      qs[2] = 0.5 * (qo[2] + Pn.w);
      qs[3] = 0.5 * (qo[3] + Pn.T);
    }
    const double sc = ft.up ? basis.inv_w_end : -basis.inv_w_end;
#pragma unroll
    for (int c = 0; c < 4; ++c) corr[ft.f][c][ft.ab] = (qs[c] - qo[c]) * sc;
  }
  __syncthreads();
  // one lane per boundary node (face node number t = tid), with that node's
  // metric terms from the boundary-node copy (fetched before the barriers)
  if (tid >= NFN) return;
  int i, j, k;
  face_node_of<N>(tid, i, j, k);
  const int n = i + NP * (j + NP * k);
  const double* const q[4] = {sq[0], sq[1], sq[2], sq[3]};
  double g[12];
  curv_gradients<N, double>(q, sD, corr, i, j, k, Ja, invJ, g);
  const double r = viscosity_ratio(ph, sq[3][n]);
  double tau[6], qT[3];
  stress64<double>(g, ph.mu * r, ph.kappa * r, tau, qT);
  const double u = sq[0][n], v = sq[1][n], w = sq[2][n];
  R* out = ffv + e * (6 * 4 * NF);
  double f[4];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int idx = d == 0 ? i : (d == 1 ? j : k);
    if (idx != 0 && idx != N) continue;
    const int ab = d == 0 ? j + NP * k : (d == 1 ? i + NP * k : i + NP * j);
    const int fi = 2 * d + (idx == N ? 1 : 0);
    contra_viscous<double>(u, v, w, tau, qT, Ja[3 * d], Ja[3 * d + 1], Ja[3 * d + 2], f);
#pragma unroll
    for (int c = 0; c < 4; ++c) out[(fi * 4 + c) * NF + ab] = static_cast<R>(f[c]);
  }
}

template <int N>
hipError_t metrics_n(const double* X, double* geo, double* geoF, bool with_f32, const DevBasis& b,
                     long long nE, int* status, hipStream_t s) {
  hipLaunchKernelGGL((k_metrics<N>), dim3(static_cast<unsigned>(nE)), dim3(CurvCfg<N>::BS), 0, s, X, geo,
                     geoF, with_f32, b, nE, status);
  return hipGetLastError();
}

template <int N, typename R>
hipError_t face_flux_curv_n(const DevMesh& m, const DevPhys& p, const DevBasis& b, const double* U,
                            void* ffv, hipStream_t s) {
  hipLaunchKernelGGL((k_face_flux_curv<N, R>), dim3(static_cast<unsigned>(m.nE)), dim3(CurvCfg<N>::BS), 0, s,
                     U, static_cast<R*>(ffv), m, p, b);
  return hipGetLastError();
}

// The right-hand side (rk = false) or RK stage (curv_line.hpp).
hipError_t launch_curv_line(int N, int precision, bool rk, const DevPhys& p, const LineLaunch& l, hipStream_t s) {
  if (precision == DG_FP64) return p.ec ? launch_curv_ec_f64(N, rk, l, s) : launch_curv_kg_f64(N, rk, l, s);
  if (p.ec && !p.mixed_ref) return hipErrorInvalidValue;  // rejected at init: needs the reference state
  return p.ec ? launch_curv_ec_f32(N, rk, l, s) : launch_curv_kg_f32(N, rk, l, s);
}

}  // namespace

hipError_t launch_metrics(int N, const double* X, double* geo, double* geoF, bool with_f32,
                          const DevBasis& b, long long nE, int* status, hipStream_t s) {
  switch (N) {
    case 3: return metrics_n<3>(X, geo, geoF, with_f32, b, nE, status, s);
    case 5: return metrics_n<5>(X, geo, geoF, with_f32, b, nE, status, s);
    case 7: return metrics_n<7>(X, geo, geoF, with_f32, b, nE, status, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_face_flux_curv(int N, int precision, const DevMesh& m, const DevPhys& p, const DevBasis& b,
                                 const double* U, void* ffv, hipStream_t s) {
  const bool f32 = precision != DG_FP64;
  switch (N) {
    case 3: return f32 ? face_flux_curv_n<3, float>(m, p, b, U, ffv, s) : face_flux_curv_n<3, double>(m, p, b, U, ffv, s);
    case 5: return f32 ? face_flux_curv_n<5, float>(m, p, b, U, ffv, s) : face_flux_curv_n<5, double>(m, p, b, U, ffv, s);
    case 7: return f32 ? face_flux_curv_n<7, float>(m, p, b, U, ffv, s) : face_flux_curv_n<7, double>(m, p, b, U, ffv, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rhs_curv(int N, int precision, const DevMesh& m, const DevPhys& p, const DevBasis& b,
                           const double* U, const void* ffv, double* Ut, int* status, hipStream_t s) {
  const Stage st{0.0, 0.0, 0.0, 0};
  return launch_curv_line(N, precision, false, p, LineLaunch{U, ffv, Ut, nullptr, status, &m, &p, &b, &st}, s);
}

hipError_t launch_rk_stage_curv(int N, int precision, const DevMesh& m, const DevPhys& p, const DevBasis& b,
                                const double* U, const void* ffv, double* G, double* U_out,
                                const Stage& st, int* status, hipStream_t s) {
  return launch_curv_line(N, precision, true, p, LineLaunch{U, ffv, G, U_out, status, &m, &p, &b, &st}, s);
}

}  // namespace dg
