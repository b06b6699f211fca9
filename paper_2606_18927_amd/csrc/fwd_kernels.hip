// Forward kernels of the split-form DGSEM operator for gfx950.
//
// Per RK stage two kernels run (paper Sec. 2.2 split-form DG on LGL nodes,
// Sec. 4 viscous fluxes and low-storage RK):
//
//   k_face_flux : U -> the normal viscous flux f_v,d (4 components) on the six
//                 face planes of every element (BR1 lifting evaluated at the
//                 face nodes only); this file;
//   k_rhs_line  : U, the neighbours' face viscous fluxes -> Ut, or the fused
//                 low-storage RK update G <- A G + dt Ut, U' <- U + B G.
//                 It recomputes its own element's lifted gradients from U
//                 (line_device.hpp).
//
// So the lifted gradients never travel through HBM: per DOF and stage the
// method moves U in twice, G in and out, U' out and three face-flux values
// (N = 7) out and in, instead of twelve gradient components out and in.
//
// Workgroup ids are remapped so that each XCD (own L2) covers one contiguous
// range of elements, keeping face neighbours in the same L2.
#include "line_device.hpp"

namespace dg {
namespace {

struct FaceArgs {
  const double* U;
  void* ffv;  // R*
  DevMesh mesh;
  DevPhys ph;
  DevBasis basis;
};
typedef const __attribute__((address_space(4))) FaceArgs* FaceArgsPtr;

__device__ inline const FaceArgs& again(FaceArgsPtr p) {
  asm volatile("" : "+s"(p));
  return *(const FaceArgs*)p;
}

// k_face_flux: f_v,d on the face planes, layout ffv[e][face][c][ab].
//
// One workgroup per element, of the line-lane shape.  A flux needs eight of the twelve
// gradient components: the normal derivatives of u, v, w, T, and of each tangential
// direction t those of u_t and of the normal velocity.
//   nodes  all lanes: (u, v, w, T) into LDS; line lanes also recover the neighbours'
//          states at the two ends of their line, the ghost values of the weak form
//          (line_device.hpp), and put the ghost velocities into LDS;
//   lines  a line lane forms the normal derivatives at its line's two ends; the other
//          wave(s) the tangential ones along the 12 (N+1) lines of the face planes,
//          two velocity components each;
//   faces  a line lane, now lane of two face nodes, forms the two fluxes; its wave
//          stores whole rows.
// What bounds it (N = 7, 32^3 elements, FP64; 0.27 ms, mixed 0.23 ms; with one lane per
// face node that read three whole lines of four fields 0.31 and 0.28 ms): HBM moves
// 1.26 GB (0.20 ms for a triad), vector instructions issue 34 % of the time (51 M wave
// instructions, before 89 M), LDS is busy 28 % (43 M cycles, before 79 M); the rest is
// the latency of the load - LDS - compute chains of the five workgroups (29 KB LDS) of a
// CU.  The sums are settled before the barriers: sunk past them they need 122 instead
// of 65 registers, and N = 5 runs 1.3x slower on half the waves.
// Mixed precision stores FP32 and computes in FP64 (without packed instructions FP32
// is no faster) with the FP32 entries of Q: their rounding is a systematic error of a
// gradient, and the two kernels' fluxes at a face have to share it, or momentum is lost
// there (with entries of D here: 5e-9 of the kinetic energy of a channel in 500 steps).
// N = 3, 48^3: 204 us, mixed 166 (207, 171); N = 5, 32^3: 153, mixed 131 (167, 142).
template <int N>
struct FaceShape {
  using L = Line<N>;
  static constexpr int TASKS = 24 * L::NP;                            // tangential lines times two components
  static constexpr int ROUNDS = (TASKS + 64 * L::FW - 1) / (64 * L::FW);
  static constexpr int OUT = 4 * L::EB;                               // tangential derivatives, 4 per face node
  // ghost velocities, 3 per face node; a single tangential wave reads all it needs
  // before it writes: they share the place of its results
  static constexpr int GHOST = L::FW == 1 ? OUT : OUT + 24 * L::NF;
  static constexpr int COUNT = L::FW == 1 ? OUT + 24 * L::NF : GHOST + 18 * L::NF;
  static constexpr int WAVES = N == 7 ? 5 : 8;                        // per SIMD, as LDS allows
};

template <int N>
__device__ __forceinline__ void face_fields(const FaceArgs& A, double* sF, int tid, const double (&u)[Line<N>::ROUNDS][5]) {
  using L = Line<N>;
#pragma unroll
  for (int r = 0; r < L::ROUNDS; ++r) {
    const unsigned n = tid + r * L::BS;
    if (n < L::NN) {
      const double* s = u[r];
      const double ir = rcp_nr(s[0]);
      const double vx = s[1] * ir, vy = s[2] * ir, vz = s[3] * ir;
      const int l = L::at(n % L::NP, (n / L::NP) % L::NP, n / L::NF);
      sF[l] = vx;
      sF[L::EB + l] = vy;
      sF[2 * L::EB + l] = vz;
      sF[3 * L::EB + l] = A.ph.gm1 * (s[4] - 0.5 * (s[1] * vx + s[2] * vy + s[3] * vz)) * A.ph.inv_R * ir;
    }
  }
}

template <int N, typename R>
__global__ __launch_bounds__(Line<N>::BS) __attribute__((amdgpu_waves_per_eu(FaceShape<N>::WAVES))) void k_face_flux(FaceArgs) {
  using L = Line<N>;
  using Fs = FaceShape<N>;
  constexpr int NP = L::NP, NF = L::NF, EB = L::EB;
  __shared__ double sF[Fs::COUNT];
  const FaceArgsPtr args = (FaceArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x;
  const int e = xcd_remap(blockIdx.x, gridDim.x);
  const FaceArgs& A = again(args);
  const long long stride = A.mesh.nE * L::NN;
  double u[L::ROUNDS][5];
  fetch_nodes<N>(A.U, stride, e, tid, u);

  if (__builtin_amdgcn_readfirstlane(tid) < 64 * L::LW) {
    const Place pl(A.mesh, e);
    const LineTask<N> t(tid);
    const bool wm = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL;
    double sn[2][5];
    bool wall[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nb = pl.neighbour(t.d, h);
      wall[h] = nb < 0;  // (there the own state)
      const unsigned o = t.end_node((h != 0) == (nb >= 0) ? 0 : N);
      const double* p = A.U + static_cast<long long>(nb >= 0 ? nb : e) * L::NN;
      sn[h][0] = p[o];
      sn[h][1] = (p + (1 + t.d) * stride)[o];
      sn[h][2] = (p + (1 + t.d1) * stride)[o];
      sn[h][3] = (p + (1 + t.d2) * stride)[o];
      sn[h][4] = (p + 4 * stride)[o];
    }
    face_fields<N>(A, sF, tid, u);
    double gh[2][4];  // ghosts: velocity along and across the line, T
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double* s = sn[h];
      const double ir = rcp_nr(s[0]);
      const double v0 = s[1] * ir, v1 = s[2] * ir, v2 = s[3] * ir;
      const double T = A.ph.gm1 * (s[4] - 0.5 * (s[1] * v0 + s[2] * v1 + s[3] * v2)) * A.ph.inv_R * ir;
      const double side = wall[h] && !wm ? -1.0 : 1.0;  // no-slip wall; the wall model's slips
      gh[h][0] = wall[h] ? -v0 : v0;
      gh[h][1] = side * v1;
      gh[h][2] = side * v2;
      gh[h][3] = wall[h] && !wm ? 2.0 * A.mesh.T_wall - T : T;
#pragma unroll
      for (int c = 0; c < 3; ++c) sF[Fs::GHOST + ((2 * t.d + h) * 3 + c) * NF + t.ab] = gh[h][c];
    }
    phase_end();

    double own[2][4], g[2][4];  // values and normal derivatives at the line's ends
    {
      const DevBasis& b = again(args).basis;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int f = c == 0 ? t.d : (c == 1 ? t.d1 : (c == 2 ? t.d2 : 3));
        double q[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) q[m] = sF[f * EB + t.node(m)];
        own[0][c] = q[0];
        own[1][c] = q[N];
        if (sizeof(R) == 4 && c == 3) {
          // the other kernel's temperatures are relative too: no row sum times T
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
    }
    phase_end();

    const FaceArgs& B = again(args);
    const double sd = (t.d == 0 ? pl.sx : (t.d == 1 ? pl.sy : pl.sz)) * B.basis.inv_w[0];
    const double s1 = t.d1 == 0 ? pl.sx : (t.d1 == 1 ? pl.sy : pl.sz);
    const double s2 = t.d2 == 0 ? pl.sx : (t.d2 == 1 ? pl.sy : pl.sz);
    const int k1 = t.d == 1 ? 2 : 0;  // tangential results of direction d1, d2
    R* out = static_cast<R*>(B.ffv) + static_cast<long long>(e) * (6 * 4 * NF);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double* o1 = &sF[Fs::OUT + ((2 * t.d + h) * 4 + k1) * NF + t.ab];
      const double* o2 = &sF[Fs::OUT + ((2 * t.d + h) * 4 + (2 - k1)) * NF + t.ab];
      double mu = B.ph.mu, kappa = B.ph.kappa;
      if (B.ph.suth) {
        const double r = viscosity_ratio(B.ph, own[h][3]);
        mu *= r;
        kappa *= r;
      }
      const double gn = sd * g[h][0];
      const double dd = (2.0 / 3.0) * (gn + s1 * o1[0] + s2 * o2[0]);
      const double t0 = mu * (gn + gn - dd);
      const double t1 = mu * (sd * g[h][1] + s1 * o1[NF]);
      const double t2 = mu * (sd * g[h][2] + s2 * o2[NF]);
      R* f = out + (2 * t.d + h) * (4 * NF);
      const unsigned ab = t.ab;
      (f + t.d * NF)[ab] = static_cast<R>(t0);
      (f + t.d1 * NF)[ab] = static_cast<R>(t1);
      (f + t.d2 * NF)[ab] = static_cast<R>(t2);
      (f + 3 * NF)[ab] = static_cast<R>(own[h][0] * t0 + own[h][1] * t1 + own[h][2] * t2 + kappa * sd * g[h][3]);
    }
  } else {
    face_fields<N>(A, sF, tid, u);
    phase_end();
    // task: the line at position pos of face 2 d + h along its first or second
    // direction t; the component u_t or u_d
    struct Task {
      int first, step, field, ghost, out, dout;
      __device__ Task(int q) {
        q = q < Fs::TASKS ? q : Fs::TASKS - 1;
        const int d = q / (8 * NP), r = q - d * (8 * NP);
        const int pos = r % NP, c = (r / NP) & 1, second = (r / (2 * NP)) & 1, h = r / (4 * NP);
        const int t = second ? (d == 2 ? 1 : 2) : (d == 0 ? 1 : 0), o = 3 - d - t;
        const int n = h ? N : 0;
        const LineTask<N> line(t, d < o ? n + NP * pos : pos + NP * n);
        first = line.first;
        step = line.step;
        field = c ? d : t;
        const int turn = field - t;  // its place in the frame of the lines along t
        ghost = Fs::GHOST + (2 * t * 3 + (turn < 0 ? turn + 3 : turn)) * NF + line.ab;
        out = Fs::OUT + ((2 * d + h) * 4 + 2 * second + c) * NF + (second ? pos : NP * pos);
        dout = second ? NP : 1;
      }
    };
    const int lane = tid - 64 * L::LW;
    double gl[Fs::ROUNDS], gr[Fs::ROUNDS];
#pragma unroll
    for (int r = 0; r < Fs::ROUNDS; ++r) {
      const Task k(lane + 64 * L::FW * r);
      gl[r] = sF[k.ghost];
      gr[r] = sF[k.ghost + 3 * NF];
    }
    if (L::FW == 1) wave_reuse();  // (the ghosts' place takes the results)
    const DevBasis& b = again(args).basis;
#pragma unroll
    for (int r = 0; r < Fs::ROUNDS; ++r) {
      const Task k(again(lane) + 64 * L::FW * r);
      double q[NP], g[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) q[m] = sF[k.field * EB + (L::SWZ ? k.first ^ (m * k.step) : k.first + m * k.step)];
      line_derivative<N, double, false>(b, q, gl[r], gr[r], g);
#pragma unroll
      for (int m = 0; m < NP; ++m) sF[k.out + m * k.dout] = b.inv_w[m] * g[m];
    }
    phase_end();
  }
}

template <int N, typename R>
hipError_t face_flux_n(const DevMesh& m, const DevPhys& p, const DevBasis& b, const double* U,
                       void* ffv, hipStream_t s) {
  FaceArgs a{U, ffv, m, p, b};
  if (sizeof(R) == 4)
    for (int i = 0; i < 16; ++i) a.basis.Q[i] = b.Qf[i];
  hipLaunchKernelGGL((k_face_flux<N, R>), dim3(static_cast<unsigned>(m.nE)), dim3(Line<N>::BS), 0, s, a);
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
