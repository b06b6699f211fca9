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
// Operator per stage (line_device.hpp has the split of the work and the weak form of
// the surface terms; k_rhs_curv is in curv_line.hpp):
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
#include "line_device.hpp"

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
    // FP32 copy of the metric terms for the mixed-precision sweeps, after the ten FP64 fields
    // (the workspace holds it only in mixed-precision contexts)
    if (with_f32) {
      float* const g32 = reinterpret_cast<float*>(geo + 10 * stride);
#pragma unroll
      for (int c = 0; c < 9; ++c) g32[c * stride + o] = static_cast<float>(Ja[c]);
    }
  }
}

// ---------------------------------------------------------- face viscous flux
// One workgroup per element, of the line-lane shape.  All twelve reference derivatives
// enter a face node's gradient:
//   nodes  all lanes: (u, v, w, T) into LDS; line lanes also the neighbours' states at the
//          two ends of their line, the ghost values of the weak form, and the metric
//          terms of their two face nodes (boundary-node copy);
//   lines  a line lane: the normal derivatives at its line's two ends, and one line of a
//          face plane for one of u, v, w, T; the other wave(s): the remaining such lines;
//   faces  a line lane, now lane of two face nodes: physical gradients, the two
//          contravariant fluxes; its wave stores whole rows.
// What bounds it (N = 7, 32^3 elements, FP64; with one lane per boundary node 0.53 ms): 0.46
// ms, 2.15 GB of HBM traffic (0.34 ms for a triad), vector instructions issue 34 % of the
// time, LDS busy 33 %; four workgroups (40 KB LDS) per CU.
// Mixed precision stores FP32 and computes in FP64 with the FP32 entries of Q, as the
// axis-aligned kernel does and for its reason.
template <int N>
struct CurvFaceShape {
  using L = Line<N>;
  static constexpr int TASKS = 48 * L::NP;                            // tangential lines times four fields
  static constexpr int MINE = 64 * L::LW;                             // of them on the line lanes
  static constexpr int ROUNDS = (TASKS - MINE + 64 * L::FW - 1) / (64 * L::FW);
  // tangential derivatives, eight per face node; before them, ghost values, four per face node
  static constexpr int OUT = 4 * L::EB, COUNT = OUT + 48 * L::NF;
  static constexpr int WAVES = 4;                                    // per SIMD
};

template <int N, typename R>
__global__ __launch_bounds__(Line<N>::BS) __attribute__((amdgpu_waves_per_eu(CurvFaceShape<N>::WAVES))) void k_face_flux_curv(
    LineArgs) {
  using L = Line<N>;
  using Fs = CurvFaceShape<N>;
  constexpr int NP = L::NP, NF = L::NF, EB = L::EB;
  __shared__ double sF[Fs::COUNT];
  const LineArgsPtr args = (LineArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x;
  const int e = xcd_remap(blockIdx.x, gridDim.x);
  // task q: the line at position pos of face 2 d + h along its first or second
  // direction t, field c
  struct Task {
    int first, step, field, ghost, out, dout;
    __device__ Task(int q) {
      q = q < Fs::TASKS ? q : Fs::TASKS - 1;
      const int d = q / (16 * NP), r = q - d * (16 * NP);
      const int pos = r % NP, c = (r / NP) & 3, second = (r / (4 * NP)) & 1, h = r / (8 * NP);
      const int t = second ? (d == 2 ? 1 : 2) : (d == 0 ? 1 : 0), o = 3 - d - t;
      const int n = h ? N : 0;
      const LineTask<N> line(t, d < o ? n + NP * pos : pos + NP * n);
      first = line.first;
      step = line.step;
      field = c;
      ghost = Fs::OUT + (2 * t * 4 + c) * NF + line.ab;
      out = Fs::OUT + ((2 * d + h) * 8 + 4 * second + c) * NF + (second ? pos : NP * pos);
      dout = second ? NP : 1;
    }
  };
  const auto along = [&](const DevBasis& b, const Task& k, double gl, double gr) {
    double q[NP], g[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) q[m] = sF[k.field * EB + (L::SWZ ? k.first ^ (m * k.step) : k.first + m * k.step)];
    if (sizeof(R) == 4) {  // (no row sum times T, as in the other kernel; the same for u, v, w)
      const double r = k.field == 3 ? q[0] : 0.0;
#pragma unroll
      for (int m = 0; m < NP; ++m) q[m] -= r;
      gl -= r;
      gr -= r;
    }
    line_derivative<N, double, false>(b, q, gl, gr, g);
#pragma unroll
    for (int m = 0; m < NP; ++m) sF[k.out + m * k.dout] = b.inv_w[m] * g[m];
  };

  double u[L::ROUNDS][5];
  {
    const LineArgs& A = again(args);
    fetch_nodes<N>(A.U, A.mesh.nE * L::NN, e, tid, u);
  }
  const auto fields = [&](const LineArgs& A) {
#pragma unroll
    for (int r = 0; r < L::ROUNDS; ++r) {
      const unsigned n = tid + r * L::BS;
      if (n < L::NN) {
        const double* s = u[r];
        const double ir = rcp_nr(s[0]);
        const double vx = s[1] * ir, vy = s[2] * ir, vz = s[3] * ir;
        const int l = L::at(n % NP, (n / NP) % NP, n / NF);
        sF[l] = vx;
        sF[EB + l] = vy;
        sF[2 * EB + l] = vz;
        sF[3 * EB + l] = A.ph.gm1 * (s[4] - 0.5 * (s[1] * vx + s[2] * vy + s[3] * vz)) * A.ph.inv_R * ir;
      }
    }
  };

  if (__builtin_amdgcn_readfirstlane(tid) < 64 * L::LW) {
    const LineArgs& A = again(args);
    const Place pl(A.mesh, e, false);
    const LineTask<N> t(tid);
    const long long stride = A.mesh.nE * L::NN;
    const int ta = t.d == 0 ? 1 : 0, tb = t.d == 2 ? 1 : 2;  // the face's first and second direction
    double sn[2][5], J[2][3][3], invJ[2];  // metric rows of d, ta, tb
    bool wall[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nb = pl.neighbour(t.d, h);
      wall[h] = nb < 0;  // (there the own state)
      const unsigned o = t.end_node((h != 0) == (nb >= 0) ? 0 : N);
      const double* p = A.U + static_cast<long long>(nb >= 0 ? nb : e) * L::NN;
#pragma unroll
      for (int v = 0; v < 5; ++v) sn[h][v] = (p + v * stride)[o];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      constexpr int NB = n_face_nodes<N>();
      const unsigned o = t.end_node(h ? N : 0), fs = static_cast<unsigned>(face_node_index<N>(o % NP, (o / NP) % NP, o / NF));
      const double* g = A.mesh.geoF + static_cast<long long>(e) * NB;
      const long long rows = A.mesh.nE * NB;
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        J[h][0][x] = (g + (3 * t.d + x) * rows)[fs];
        J[h][1][x] = (g + (3 * ta + x) * rows)[fs];
        J[h][2][x] = (g + (3 * tb + x) * rows)[fs];
      }
      invJ[h] = (g + 9 * rows)[fs];
    }
    fields(A);
    double gh[2][4];  // ghosts: u, v, w, T
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double* s = sn[h];
      const double ir = rcp_nr(s[0]);
      const double v0 = s[1] * ir, v1 = s[2] * ir, v2 = s[3] * ir;
      const double T = A.ph.gm1 * (s[4] - 0.5 * (s[1] * v0 + s[2] * v1 + s[3] * v2)) * A.ph.inv_R * ir;
      const double side = wall[h] ? -1.0 : 1.0;  // isothermal no-slip wall
      gh[h][0] = side * v0;
      gh[h][1] = side * v1;
      gh[h][2] = side * v2;
      gh[h][3] = wall[h] ? 2.0 * A.mesh.T_wall - T : T;
#pragma unroll
      for (int c = 0; c < 4; ++c) sF[Fs::OUT + ((2 * t.d + h) * 4 + c) * NF + t.ab] = gh[h][c];
    }
    phase_end();
    double gl, gr;
    {
      const Task k(again(tid));
      gl = sF[k.ghost];
      gr = sF[k.ghost + 4 * NF];
    }
    phase_end();

    double own[2][4], g[2][4];  // values and normal derivatives at the line's ends
    const DevBasis& b = again(args).basis;
    along(b, Task(again(tid)), gl, gr);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double q[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) q[m] = sF[c * EB + t.node(m)];
      own[0][c] = q[0];
      own[1][c] = q[N];
      if (sizeof(R) == 4 && c == 3) {
#pragma unroll
        for (int m = 0; m < NP; ++m) q[m] -= own[0][3];
        gh[0][3] -= own[0][3];
        gh[1][3] -= own[0][3];
      }
      g[0][c] = g[1][c] = 0.0;
#pragma unroll
      for (int m = N; m > 0; --m) g[0][c] += q_im<N, double>(b, 0, m) * q[m];
#pragma unroll
      for (int m = 0; m < N; ++m) g[1][c] -= q_im<N, double>(b, m, N) * q[m];
      g[0][c] -= 0.5 * gh[0][c];
      g[1][c] += 0.5 * gh[1][c];
      if (c & 1) settle(g);
    }
    phase_end();

    const LineArgs& B = again(args);
    const double iw = B.basis.inv_w[0];
    R* out = static_cast<R*>(const_cast<void*>(B.ffv)) + static_cast<long long>(e) * (6 * 4 * NF);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double* o = &sF[Fs::OUT + (2 * t.d + h) * 8 * NF + t.ab];
      double gp[12];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double gn = invJ[h] * iw * g[h][c], ga = invJ[h] * o[c * NF], gb = invJ[h] * o[(4 + c) * NF];
#pragma unroll
        for (int x = 0; x < 3; ++x) gp[3 * c + x] = J[h][0][x] * gn + J[h][1][x] * ga + J[h][2][x] * gb;
      }
      const double r = viscosity_ratio(B.ph, own[h][3]);
      double tau[6], qT[3], f[4];
      stress64<double>(gp, B.ph.mu * r, B.ph.kappa * r, tau, qT);
      contra_viscous<double>(own[h][0], own[h][1], own[h][2], tau, qT, J[h][0][0], J[h][0][1], J[h][0][2], f);
      R* dst = out + (2 * t.d + h) * (4 * NF);
#pragma unroll
      for (int c = 0; c < 4; ++c) (dst + c * NF)[static_cast<unsigned>(t.ab)] = static_cast<R>(f[c]);
    }
  } else {
    fields(again(args));
    phase_end();
    const int lane = tid - 64 * L::LW;
    double gl[Fs::ROUNDS], gr[Fs::ROUNDS];
#pragma unroll
    for (int r = 0; r < Fs::ROUNDS; ++r) {
      const Task k(Fs::MINE + lane + 64 * L::FW * r);
      gl[r] = sF[k.ghost];
      gr[r] = sF[k.ghost + 4 * NF];
    }
    phase_end();
    const DevBasis& b = again(args).basis;
#pragma unroll
    for (int r = 0; r < Fs::ROUNDS; ++r) along(b, Task(Fs::MINE + again(lane) + 64 * L::FW * r), gl[r], gr[r]);
    phase_end();
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
  LineArgs a{U, ffv, nullptr, nullptr, nullptr, m, p, b, Stage{}};
  if (sizeof(R) == 4)
    for (int i = 0; i < 16; ++i) a.basis.Q[i] = b.Qf[i];
  hipLaunchKernelGGL((k_face_flux_curv<N, R>), dim3(static_cast<unsigned>(m.nE)), dim3(Line<N>::BS), 0, s, a);
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
