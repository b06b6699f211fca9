// Forward kernels of the split-form DGSEM operator for gfx950.
//
// Per RK stage two kernels run (paper Sec. 2.2 split-form DG on LGL nodes,
// Sec. 4 viscous fluxes and low-storage RK):
//
//   k_face_flux : U -> the normal viscous flux f_v,d (4 components) on the six
//                 face planes of every element (BR1 lifting evaluated at the
//                 face nodes only);
//   k_rhs_line  : U, the neighbours' face viscous fluxes -> Ut, or the fused
//                 low-storage RK update G <- A G + dt Ut, U' <- U + B G.
//                 It recomputes its own element's lifted gradients from U.
//
// So the lifted gradients never travel through HBM: per DOF and stage the
// method moves U in twice, G in and out, U' out and three face-flux values
// (N = 7) out and in, instead of twelve gradient components out and in.
//
// This file holds the first kernel; the second is in line_device.hpp.
//
// Mixed precision (R = float): the LDS fields, gradients and viscous fluxes are
// FP32; the primitive recovery and the lifting corrections stay FP64.
// Temperature is stored relative to the element's first node, with the difference
// taken in FP64.
//
// Workgroup ids are remapped so that each XCD (own L2) covers one contiguous
// range of elements, keeping face neighbours in the same L2.
#include "dg_device.hpp"

namespace dg {
namespace {

// Vector of two R values (one 64- or 128-bit LDS access).
template <typename R>
struct V2T;
template <>
struct V2T<double> {
  using type = double2;
};
template <>
struct V2T<float> {
  using type = float2;
};

// Line sums sum_m Q_im q_m, Q = diag(w) D, along direction d of (u, v, w, T) held as
// LDS pairs q[0] = (u, v), q[1] = (w, T) at node (i, j, k); Q is read once per line
// position.
template <int N, typename R, int d, typename V2>
__device__ inline void line_sums_pairs(const R* sQ, const V2 (*q)[Geo<N>::EB], int i, int j, int k,
                                       R a[4]) {
  using Gm = Geo<N>;
  constexpr int NP = Gm::NP;
  const int idx = d == 0 ? i : (d == 1 ? j : k);
  a[0] = a[1] = a[2] = a[3] = R(0);
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    const int lm = d == 0 ? Gm::lds(m, j, k) : (d == 1 ? Gm::lds(i, m, k) : Gm::lds(i, j, m));
    const R Qm = sQ[idx * Gm::DS + m];
    const V2 uv = q[0][lm], wT = q[1][lm];
    a[0] += Qm * uv.x;
    a[1] += Qm * uv.y;
    a[2] += Qm * wT.x;
    a[3] += Qm * wT.y;
  }
}

// BR1 lifted gradients g[3 q + d] of (u, v, w, T) (LDS pairs) at node
// (i, j, k), with the lifting corrections ssq of the six faces; sx, sy, sz include the
// nodes' 1 / w.  The entries of Q are those of the line-lane kernel: the rounding
// of a row's entries is a systematic error of a gradient (the row sum, times the mean
// velocity), and in mixed precision the two kernels' fluxes at a face have to share it,
// or momentum is lost there (5e-9 of the channel's kinetic energy in 500 steps).
template <int N, typename R, typename V2>
__device__ inline void lifted_gradients(const R* sQ, const V2 (*q)[Geo<N>::EB],
                                        const R (*ssq)[4][Geo<N>::NF], int i, int j, int k, R sx,
                                        R sy, R sz, R g[12]) {
  constexpr int NP = N + 1;
  R a[4];
  line_sums_pairs<N, R, 0, V2>(sQ, q, i, j, k, a);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (i == 0) a[c] += ssq[0][c][j + NP * k];
    if (i == N) a[c] += ssq[1][c][j + NP * k];
    g[3 * c + 0] = sx * a[c];
  }
  line_sums_pairs<N, R, 1, V2>(sQ, q, i, j, k, a);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (j == 0) a[c] += ssq[2][c][i + NP * k];
    if (j == N) a[c] += ssq[3][c][i + NP * k];
    g[3 * c + 1] = sy * a[c];
  }
  line_sums_pairs<N, R, 2, V2>(sQ, q, i, j, k, a);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (k == 0) a[c] += ssq[4][c][i + NP * j];
    if (k == N) a[c] += ssq[5][c][i + NP * j];
    g[3 * c + 2] = sz * a[c];
  }
}

// Per-element reference (p, e, T) of the mixed-precision sweeps: the values at
// node 0 (state s0), or zero in FP64 and with the subtraction switched off.
template <typename R>
__device__ inline bool uses_ref(const DevPhys& ph) {
  return sizeof(R) == sizeof(float) && ph.mixed_ref;
}

template <typename R>
__device__ inline void element_ref(const double s0[5], const DevPhys& ph, double& p_ref,
                                   double& e_ref, double& T_ref) {
  if (!uses_ref<R>(ph)) {
    p_ref = e_ref = T_ref = 0.0;
    return;
  }
  const Prim P = primitives(s0, ph);
  p_ref = P.p;
  e_ref = P.e;
  T_ref = P.T;
}

// --------------------------------------------------------------------------
// k_face_flux: f_v,d on the face planes, layout ffv[e][face][c][ab]
// --------------------------------------------------------------------------
template <int N, typename R>
__global__ __launch_bounds__(Cfg<N>::BS) __attribute__((amdgpu_waves_per_eu(Cfg<N>::FACE_WAVES))) void k_face_flux(
    const double* __restrict__ U, R* __restrict__ ffv, DevMesh mesh, DevPhys ph, DevBasis basis) {
  using Gm = Geo<N>;
  constexpr int NP = Gm::NP, NF = Gm::NF, NN = Gm::NN, EB = Gm::EB;
  constexpr int EPB = Cfg<N>::EPB, BS = Cfg<N>::BS;
  constexpr int NFN = n_face_nodes<N>();
  static_assert(EPB * NFN <= BS, "one lane per face node");
  using V2 = typename V2T<R>::type;
  __shared__ R sQ[NP * Gm::DS];
  __shared__ double sW[NP];  // 1 / w_i
  __shared__ V2 sq[EPB][2][EB];  // (u, v), (w, T - T_ref)
  __shared__ R ssq[EPB][6][4][NF];
  constexpr bool MIXED = sizeof(R) == 4;
  // mixed precision: the FP64 (u, v, w, T) of every node, for the lifting terms
  __shared__ double sqd[MIXED ? EPB : 1][4][MIXED ? NN : 1];

  const int tid = threadIdx.x;
  const long long nE = mesh.nE;
  const long long stride = nE * NN;
  const long long e0 = static_cast<long long>(xcd_remap(blockIdx.x, gridDim.x)) * EPB;
  int ex0 = 0, ey0 = 0, ez0 = 0;
  elem_coords(e0 < nE ? e0 : 0, mesh, ex0, ey0, ez0);

  // P1: node lanes stage (u, v, w, T - T_ref) in LDS (and, in mixed
  // precision, an FP64 copy of (u, v, w, T)); face lanes fetch the
  // neighbour state and form the BR1 lifting corrections in FP64 after the
  // barrier, with the own values from LDS
  const bool face_lane = tid < n_face_tasks<N>();
  const bool face_ok = face_lane && (EPB == 1 ? e0 : e0 + FaceTask<N>(face_lane ? tid : 0).le) < nE;
  // the own state is fetched first, so that it and the neighbour's face node
  // are in flight together
  const int nle = EPB == 1 ? 0 : tid / NN;
  const int node = tid - nle * NN;
  const long long ne = EPB == 1 ? e0 : e0 + nle;
  const bool node_ok = (EPB == 1 ? tid < NN : nle < EPB) && ne < nE;
  double s[5] = {1.0, 0.0, 0.0, 0.0, 1.0}, s0[5] = {1.0, 0.0, 0.0, 0.0, 1.0};
  if (node_ok) {
    load_state(U, stride, ne * NN + node, s);
    if (uses_ref<R>(ph)) load_state(U, stride, ne * NN, s0);
  }
  double sn[5] = {1.0, 0.0, 0.0, 0.0, 1.0};
  bool fwall = true;
  if (face_ok) {
    const FaceTask<N> ft(tid);
    const long long te = EPB == 1 ? e0 : e0 + ft.le;
    int ex = ex0, ey = ey0, ez = ez0;
    if (EPB > 1) elem_coords(te, mesh, ex, ey, ez);
    const long long nb = neighbour(mesh, ex, ey, ez, ft.d, ft.up);
    fwall = nb < 0;
    if (!fwall) load_state(U, stride, nb * NN + ft.nb_node(), sn);
  }
  if (node_ok) {
    const int i = node % NP, j = (node / NP) % NP, k = node / NF;
    const Prim P = primitives(s, ph);
    double p_ref, e_ref, T_ref;
    element_ref<R>(s0, ph, p_ref, e_ref, T_ref);
    const int l = Gm::lds(i, j, k);
    sq[nle][0][l] = V2{static_cast<R>(P.u), static_cast<R>(P.v)};
    sq[nle][1][l] = V2{static_cast<R>(P.w), static_cast<R>(P.T - T_ref)};
    if (MIXED) {
      sqd[nle][0][node] = P.u;
      sqd[nle][1][node] = P.v;
      sqd[nle][2][node] = P.w;
      sqd[nle][3][node] = P.T;
    }
  }
  static_assert(NP * NP <= BS, "one lane per entry of Q");
  if (tid < NP * NP) {
    const int i = tid / NP, m = tid % NP;
    const bool flip = i + m > N;  // Q_im = -Q_mi = -Q_(N-i)(N-m): the entries 0 <= i < m <= N - i are stored
    const int a = flip ? (i < m ? N - m : N - i) : (i < m ? i : m), c = flip ? (i < m ? N - i : N - m) : (i < m ? m : i);
    R q = i == m ? (i == 0 ? R(-0.5) : (i == N ? R(0.5) : R(0))) : R(0);
    if (i != m) {
      const int id = a * N - a * (a - 1) + c - a - 1;
#pragma unroll
      for (int t = 0; t < (NP * NP) / 4; ++t) {
        const R b = sizeof(R) == 4 ? static_cast<R>(basis.Qf[t]) : static_cast<R>(basis.Q[t]);
        q = id == t ? b : q;
      }
      if (i > m) q = -q;
    }
    sQ[i * Gm::DS + m] = q;
    if (m == 0) {
      double w = basis.inv_w[0];
#pragma unroll
      for (int t = 1; t < NP; ++t) w = i == t ? basis.inv_w[t] : w;
      sW[i] = w;
    }
  }
  __syncthreads();
  {
    if (face_ok) {
      const FaceTask<N> ft(tid);
      double qo[4];
      if (MIXED) {
        const int on = ft.own_node();
#pragma unroll
        for (int c = 0; c < 4; ++c) qo[c] = sqd[ft.le][c][on];
      } else {
        const int lo = Gm::lds(ft.oi, ft.oj, ft.ok);
        const V2 uv = sq[ft.le][0][lo], wT = sq[ft.le][1][lo];
        qo[0] = uv.x;
        qo[1] = uv.y;
        qo[2] = wT.x;
        qo[3] = wT.y;
      }
      double qs[4];
      wall_lifting_value(mesh, ft.d, qo, qs);
      if (!fwall) {
        const Prim Pn = primitives(sn, ph);
        qs[0] = 0.5 * (qo[0] + Pn.u);
        qs[1] = 0.5 * (qo[1] + Pn.v);
        qs[2] = 0.5 * (qo[2] + Pn.w);
        qs[3] = 0.5 * (qo[3] + Pn.T);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) ssq[ft.le][ft.f][c][ft.ab] = static_cast<R>(ft.up ? qs[c] - qo[c] : qo[c] - qs[c]);
    }
    __syncthreads();
  }

  // P2: one lane per face node: lifted gradients and f_v,d of each face the
  // node lies on
  const int le = EPB == 1 ? 0 : tid / NFN;
  const long long e = EPB == 1 ? e0 : e0 + le;
  if ((EPB == 1 ? tid < NFN : le < EPB) && e < nE) {
    int i, j, k;
    face_node_of<N>(tid - le * NFN, i, j, k);
    int ex = ex0, ey = ey0, ez = ez0;
    if (EPB > 1) elem_coords(e, mesh, ex, ey, ez);
    R g[12];
    lifted_gradients<N, R, V2>(sQ, sq[le], ssq[le], i, j, k, static_cast<R>(mesh.s[0][ex] * sW[i]),
                               static_cast<R>(mesh.s[1][ey] * sW[j]), static_cast<R>(mesh.s[2][ez] * sW[k]), g);
    const int l = Gm::lds(i, j, k);
    const V2 uv = sq[le][0][l], wT = sq[le][1][l];
    const R u = uv.x, v = uv.y, w = wT.x;
    R mu = static_cast<R>(ph.mu), kappa = static_cast<R>(ph.kappa);
    if (ph.suth) {
      // mu(T) at the node's temperature: in FP64 the LDS holds T itself, in
      // mixed precision the FP64 copy holds it
      const double T = MIXED ? sqd[le][3][i + NP * (j + NP * k)] : static_cast<double>(wT.y);
      const R r = static_cast<R>(viscosity_ratio(ph, T));
      mu *= r;
      kappa *= r;
    }
    R* out = ffv + e * (6 * 4 * NF);
    R f[4];
    if (i == 0 || i == N) {
      viscous_flux<0, R>(u, v, w, g, mu, kappa, f);
      const int fi = i == 0 ? 0 : 1;
#pragma unroll
      for (int c = 0; c < 4; ++c) out[(fi * 4 + c) * NF + j + NP * k] = f[c];
    }
    if (j == 0 || j == N) {
      viscous_flux<1, R>(u, v, w, g, mu, kappa, f);
      const int fi = j == 0 ? 2 : 3;
#pragma unroll
      for (int c = 0; c < 4; ++c) out[(fi * 4 + c) * NF + i + NP * k] = f[c];
    }
    if (k == 0 || k == N) {
      viscous_flux<2, R>(u, v, w, g, mu, kappa, f);
      const int fi = k == 0 ? 4 : 5;
#pragma unroll
      for (int c = 0; c < 4; ++c) out[(fi * 4 + c) * NF + i + NP * j] = f[c];
    }
  }
}

template <int N, typename R>
hipError_t face_flux_n(const DevMesh& m, const DevPhys& p, const DevBasis& b, const double* U,
                       void* ffv, hipStream_t s) {
  hipLaunchKernelGGL((k_face_flux<N, R>), dim3(n_blocks<N>(m.nE)), dim3(Cfg<N>::BS), 0, s, U,
                     static_cast<R*>(ffv), m, p, b);
  return hipGetLastError();
}

// The right-hand side (rk = false) or RK stage with line lanes.
hipError_t launch_line(int N, int precision, bool rk, const DevPhys& p, const LineLaunch& l, hipStream_t s) {
  if (precision == DG_FP64) return p.ec ? launch_line_ec_f64(N, rk, l, s) : launch_line_kg_f64(N, rk, l, s);
  if (p.ec && !p.mixed_ref) return hipErrorInvalidValue;  // rejected at init: needs the reference state
  return p.ec ? launch_line_ec_f32(N, rk, l, s) : launch_line_kg_f32(N, rk, l, s);
}

}  // namespace

hipError_t launch_face_flux(int N, int precision, const DevMesh& m, const DevPhys& p,
                            const DevBasis& b, const double* U, void* ffv, hipStream_t s) {
  if (m.nE <= 0 || !p.viscous) return hipSuccess;
  const bool f32 = precision != DG_FP64;
  switch (N) {
    case 3: return f32 ? face_flux_n<3, float>(m, p, b, U, ffv, s) : face_flux_n<3, double>(m, p, b, U, ffv, s);
    case 5: return f32 ? face_flux_n<5, float>(m, p, b, U, ffv, s) : face_flux_n<5, double>(m, p, b, U, ffv, s);
    case 7: return f32 ? face_flux_n<7, float>(m, p, b, U, ffv, s) : face_flux_n<7, double>(m, p, b, U, ffv, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rhs(int N, int precision, const DevMesh& m, const DevPhys& p,
                      const DevBasis& b, const double* U, const void* ffv, double* Ut,
                      int* status, hipStream_t s) {
  if (m.nE <= 0) return hipSuccess;
  const Stage st{0.0, 0.0, 0.0, 0};
  return launch_line(N, precision, false, p, LineLaunch{U, ffv, Ut, nullptr, status, &m, &p, &b, &st}, s);
}

hipError_t launch_rk_stage(int N, int precision, const DevMesh& m, const DevPhys& p,
                           const DevBasis& b, const double* U, const void* ffv, double* G,
                           double* U_out, const Stage& st, int* status, hipStream_t s) {
  if (m.nE <= 0) return hipSuccess;
  return launch_line(N, precision, true, p, LineLaunch{U, ffv, G, U_out, status, &m, &p, &b, &st}, s);
}

}  // namespace dg
