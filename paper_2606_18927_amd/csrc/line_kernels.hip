// Right-hand side (and fused RK stage) with line lanes, for gfx950 (FP64,
// Kennedy-Gruber / Lax-Friedrichs pair).
//
// What bounds it (N = 7, 32^3 elements; counters of the RK instance): vector
// instructions issue 47 % of the time (225 M wave instructions, 163 M of them
// FP64; with one lane per node and every node reading its lines from LDS the
// same stage took 0.98 ms and its LDS was busy 55 % of the time, here 0.78 ms and
// 25 %), HBM moves 3.4 GB; a CU holds two workgroups (74 KB LDS, 252 registers: the
// whole line and its sums), so eight waves have to hide each other's LDS and
// barrier latencies.
//
// One workgroup works on one element at a time.  Two kinds of phases alternate,
// with the nodal fields in LDS between them:
//
//   node phases  one lane per node: recover the primitives of U; lifted velocity
//                gradients -> viscous fluxes; sum the three directions and write
//                Ut or update G and U'.
//   line phases  one lane per grid line of the element (3 (N+1)^2 lines).  The whole
//                line's values sit in the lane's registers, so each is read from
//                LDS once per direction instead of once per node and line position,
//                the coefficients are scalar operands, and a symmetric two-point
//                flux is evaluated once per pair of nodes (N (N+1) / 2 instead of
//                (N+1)^2 evaluations per line).  The workgroup's other wave(s) take
//                the face nodes of the lines' ends and the diffusive part of the
//                energy meanwhile, which makes the waves' shares about equal.
//
// A line lane works in its own frame: the velocity along the line first, then
// the two others in cyclic order, so one code serves the three directions.
//
// Summation by parts does the surface terms.  With Q = diag(w) D, Q antisymmetric
// but for Q_00 = -Q_NN = -1/2, the strong form of every term
//   sum_m D_im q_m + (delta_iN (q* - q_N) - delta_i0 (q* - q_0)) / w_i,  q* = (q + q_ghost) / 2,
// is (1 / w_i) (sum_{m != i} Q_im q_m + (delta_iN - delta_i0) q_ghost / 2): the own
// end value cancels and the neighbour's face value is one more point of the
// line.  The same holds for the two-point fluxes (the surface flux's central
// part is the two-point flux of the two sides).  A wall is a ghost value too:
// 2 q* - q for a lifted quantity or a viscous flux with wall value q*, and the
// mirrored velocity for the pressure-only convective flux (its mass flux is
// exactly zero).
#include "dg_device.hpp"

namespace dg {
namespace {

// Shape of a workgroup and of its LDS fields.  x-rows of 2^n nodes are
// xor-swizzled twice (node i of row j of plane k at slot i ^ j of row j ^ k), so
// that the 64-bit accesses of line lanes and of node lanes meet no bank
// conflicts in any direction; rows of 6 are padded to 7.
template <int N>
struct Line {
  static constexpr int NP = N + 1, NF = NP * NP, NN = NF * NP;
  static constexpr bool SWZ = (NP & (NP - 1)) == 0;
  static constexpr int RS = SWZ ? NP : NP + 1;
  static constexpr int EB = RS * NP * NP;
  static constexpr int LINES = 3 * NF;
  static constexpr int LW = (LINES + 63) / 64;          // line waves
  static constexpr int FW = N == 5 ? 2 : 1;             // face waves
  static constexpr int BS = 64 * (LW + FW);
  static constexpr int ROUNDS = (NN + BS - 1) / BS;     // of the node phases
  // a direction's lines fill whole waves: the direction is wave-uniform
  static constexpr bool UNIFORM = NF == 64;
  static constexpr int FL = UNIFORM ? 3 : 1;            // lines of a face lane
  // fields: halves of rho, u, v, w, p, e (0..5) and T (6); raw velocity gradients
  // 7 + 3 q + d, then the half viscous fluxes (tau_00, tau_11, tau_22, tau_01,
  // tau_02, tau_12, u . tau_d); at the end the directions' sums (0..14) and their
  // diffusive energy parts (15..17); last mu(T) / mu (Sutherland's law only).  The 8 values of each of the 2 LINES line
  // ends take, where a wave holds one direction, the gradient fields that this
  // wave alone writes after reading them, else a region of their own.
  static constexpr int ENDS = 18 * EB;
  static constexpr int MU = UNIFORM ? 18 * EB : ENDS + 16 * LINES;
  __device__ static int end_at(int d, int k, int ab) {
    return UNIFORM ? (7 + 3 * (k >> 3) + d) * EB + (k & 7) * NF + ab : ENDS + k * LINES + d * NF + ab;
  }
  __device__ static constexpr int at(int i, int j, int k) {
    return SWZ ? (i ^ j) + NP * (j ^ k) + NF * k : i + RS * (j + NP * k);
  }
};

template <int N>
inline size_t line_lds(const DevPhys& p) {
  return sizeof(double) * (static_cast<size_t>(Line<N>::MU) + (p.viscous && p.suth ? Line<N>::EB : 0) + N + 1);
}

// Arguments of the kernel.  The kernel reads them from the kernel-argument
// segment where a phase needs them, instead of holding all of them (the
// coefficients among them) in scalar registers from the start.
struct LineArgs {
  const double* U;
  const double* ffv;
  double* out;
  double* U_out;
  int* status;
  DevMesh mesh;
  DevPhys ph;
  DevBasis basis;
  Stage st;
};
typedef const __attribute__((address_space(4))) LineArgs* LineArgsPtr;

__device__ inline const LineArgs& again(LineArgsPtr p) {
  asm volatile("" : "+s"(p));
  return *(const LineArgs*)p;
}

// A lane index whose derived values are formed again after this point instead of
// being held in registers across the phases before it.
__device__ inline int again(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Q_im for i < m (DevBasis), a scalar operand.
template <int N>
__device__ inline double q_im(const DevBasis& b, int i, int m) {
  const int a = i + m > N ? N - m : i, c = i + m > N ? N - i : m;
  return b.Q[a * N - a * (a - 1) + c - a - 1];
}

// g_i = sum_{m != i} Q_im q_m plus the two ghost values.
template <int N>
__device__ inline void line_derivative(const DevBasis& b, const double (&q)[N + 1], double ghost_lo, double ghost_hi,
                                       double (&g)[N + 1]) {
#pragma unroll
  for (int i = 0; i <= N; ++i) g[i] = 0.0;
  g[0] = -0.5 * ghost_lo;
  g[N] = 0.5 * ghost_hi;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int m = i + 1; m <= N; ++m) {
      const double c = q_im<N>(b, i, m);
      g[i] += c * q[m];
      g[m] -= c * q[i];
    }
}

// sqrt(x) for x > 0 of moderate size: the hardware estimate of 1 / sqrt(x) and
// one coupled and one residual Newton step.
__device__ inline double sqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}

// The line of a line lane: direction d, position ab in the face
// plane, and the LDS entries of its nodes.
template <int N>
struct LineTask {
  static constexpr int NP = N + 1, NF = NP * NP;
  int d, ab, d1, d2, first, step;
  // line t of the element; lanes beyond the last line take the last one too (and
  // write the same values to the same places)
  __device__ explicit LineTask(int t)
      : LineTask(Line<N>::UNIFORM ? __builtin_amdgcn_readfirstlane(static_cast<unsigned>(t) / NF) : clamped(t) / NF,
                 clamped(t) % NF) {}
  __device__ static unsigned clamped(int t) { return Line<N>::UNIFORM || t < Line<N>::LINES ? t : Line<N>::LINES - 1; }
  __device__ LineTask(int d_, int ab_) : d(d_), ab(ab_) {
    d1 = d == 2 ? 0 : d + 1;  // the two other directions, cyclic
    d2 = d == 0 ? 2 : d - 1;
    const int a = static_cast<unsigned>(ab) % NP, b = static_cast<unsigned>(ab) / NP;
    first = d == 0 ? Line<N>::at(0, a, b) : (d == 1 ? Line<N>::at(a, 0, b) : Line<N>::at(a, b, 0));
    step = Line<N>::SWZ ? (d == 0 ? 1 : (d == 1 ? NP + 1 : NF + NP)) : (d == 0 ? 1 : (d == 1 ? Line<N>::RS : Line<N>::RS * NP));
  }
  // node m of the line (the swizzle is linear over xor)
  __device__ int node(int m) const { return Line<N>::SWZ ? first ^ (m * step) : first + m * step; }
  // global index of its first (m = 0) or last (m = N) node in the element
  __device__ unsigned end_node(int m) const {
    const unsigned a = static_cast<unsigned>(ab) % NP, b = static_cast<unsigned>(ab) / NP;
    return d == 0 ? m + NP * a + NF * b : (d == 1 ? a + NP * m + NF * b : a + NP * b + NF * m);
  }
};

// An element's position, formed once per element: coordinates, and neighbour
// across the face 2 d + h (-1 on a wall).
struct Place {
  int ex, ey, ez, nb[6];
  double sx, sy, sz;
  __device__ Place(const DevMesh& m, int e) {
    elem_coords(e, m, ex, ey, ez);
    ex = __builtin_amdgcn_readfirstlane(ex);
    ey = __builtin_amdgcn_readfirstlane(ey);
    ez = __builtin_amdgcn_readfirstlane(ez);
    const int sxy = m.n[0] * m.n[1];
    nb[0] = ex > 0 ? e - 1 : (m.bc[0] == DG_BC_PERIODIC ? e + m.n[0] - 1 : -1);
    nb[1] = ex < m.n[0] - 1 ? e + 1 : (m.bc[0] == DG_BC_PERIODIC ? e - m.n[0] + 1 : -1);
    nb[2] = ey > 0 ? e - m.n[0] : (m.bc[1] == DG_BC_PERIODIC ? e + sxy - m.n[0] : -1);
    nb[3] = ey < m.n[1] - 1 ? e + m.n[0] : (m.bc[1] == DG_BC_PERIODIC ? e - sxy + m.n[0] : -1);
    nb[4] = ez > 0 ? e - sxy : (m.bc[2] == DG_BC_PERIODIC ? e + sxy * (m.n[2] - 1) : -1);
    nb[5] = ez < m.n[2] - 1 ? e + sxy : (m.bc[2] == DG_BC_PERIODIC ? e - sxy * (m.n[2] - 1) : -1);
    // (scalar loads: the tables are constant while the kernel runs)
    typedef const __attribute__((address_space(4))) double* Table;
    sx = ((Table)(uintptr_t)m.s[0])[ex];
    sy = ((Table)(uintptr_t)m.s[1])[ey];
    sz = ((Table)(uintptr_t)m.s[2])[ez];
  }
  __device__ int neighbour(int d, int h) const {
    return h ? pick3(nb[1], nb[3], nb[5], d) : pick3(nb[0], nb[2], nb[4], d);
  }
};

// The fetches below are unconditional: a lane without a node, or a face without a
// neighbour, reads a valid address it has no use for.  A load under a condition is
// waited for where the condition ends (its register is merged with another
// value's), and would not be in flight over the phases after it.
template <int N>
__device__ inline unsigned node_of(int tid, int r) {
  const unsigned n = tid + r * Line<N>::BS;
  return Line<N>::NN % Line<N>::BS == 0 || n < Line<N>::NN ? n : 0;
}

template <int N>
__device__ inline void fetch_nodes(const double* __restrict__ U, long long stride, int e, int tid,
                                   double (&u)[Line<N>::ROUNDS][5]) {
  using L = Line<N>;
#pragma unroll
  for (int r = 0; r < L::ROUNDS; ++r)
#pragma unroll
    for (int v = 0; v < 5; ++v) u[r][v] = (U + v * stride + static_cast<long long>(e) * L::NN)[node_of<N>(tid, r)];
}

// Line q of a face lane (q < FL).
template <int N>
__device__ inline LineTask<N> face_line(int lane, int q) {
  if constexpr (Line<N>::UNIFORM)
    return LineTask<N>(q, lane);
  else
    return LineTask<N>(lane);
}

// The neighbours' states at the ends h of the face lane's lines q, in the line frame
// (rho, momentum along the line and across, E).
template <int N>
__device__ inline void fetch_faces(const double* __restrict__ U, long long stride, const Place& pl, int e, int lane,
                                   double (&sn)[Line<N>::FL][2][5]) {
  using L = Line<N>;
#pragma unroll
  for (int q = 0; q < L::FL; ++q) {
    const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nb = pl.neighbour(t.d, h);
      const unsigned o = t.end_node(h ? 0 : N);
      const double* s = U + static_cast<long long>(nb >= 0 ? nb : e) * L::NN;
      sn[q][h][0] = s[o];
      sn[q][h][1] = (s + (1 + t.d) * stride)[o];
      sn[q][h][2] = (s + (1 + t.d1) * stride)[o];
      sn[q][h][3] = (s + (1 + t.d2) * stride)[o];
      sn[q][h][4] = (s + 4 * stride)[o];
    }
  }
}

// Values that have to exist at this point: the compiler would else sink the sums
// that make them into a later phase, and hold all their operands until then.
template <int A, int B>
__device__ __forceinline__ void settle(double (&x)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) asm volatile("" : "+v"(x[a][b]));
}

// A phase boundary: a workgroup barrier that no instruction is scheduled across
// (the phases' values would else overlap and spill).
__device__ __forceinline__ void phase_end() {
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
}

// Node phase: primitives of the states u into the LDS fields.
template <int N, bool VISC>
__device__ __forceinline__ void primitives_to_lds(const LineArgs& A, double* const sF, const int tid,
                                             const double (&u)[Line<N>::ROUNDS][5]) {
  using L = Line<N>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, ROUNDS = L::ROUNDS;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const unsigned n = tid + r * L::BS;
    if (n < NN) {
      const double* s = u[r];
      const double ir = rcp_nr(s[0]);
      const double vx = s[1] * ir, vy = s[2] * ir, vz = s[3] * ir;
      const double p = A.ph.gm1 * (s[4] - 0.5 * s[0] * (vx * vx + vy * vy + vz * vz));
      const double T = p * A.ph.inv_R * ir;
      if (!(s[0] > 0.0) || !(p > 0.0)) A.status[0] = 1;
      const int l = L::at(n % NP, (n / NP) % NP, n / NF);
      sF[l] = 0.5 * s[0];
      sF[EB + l] = 0.5 * vx;
      sF[2 * EB + l] = 0.5 * vy;
      sF[3 * EB + l] = 0.5 * vz;
      sF[4 * EB + l] = 0.5 * p;
      sF[5 * EB + l] = 0.5 * (s[4] * ir);
      sF[6 * EB + l] = T;
      if (VISC && A.ph.suth) sF[L::MU + l] = viscosity_ratio(A.ph, T);
    }
  }
}

// The phases of a workgroup as its face waves (FACE) or line waves run them: the two
// run the same node phases and meet at the same barriers.  tid: the lane's number
// in the node phases; wtid: its line (>= 64 LW: face lane).
template <int N, bool RK, bool VISC, bool FACE>
__device__ __forceinline__ void rhs_line_phases(const LineArgsPtr args, double* const lds, int e, const int step_e,
                                               const int end_e, const int tid, const int wtid) {
  using L = Line<N>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, BS = L::BS, ROUNDS = L::ROUNDS, FL = L::FL;
  constexpr bool PERSIST = N == 7;
  double* const sW = lds;
  double* const sF = lds + NP;
  double u[ROUNDS][5];
  double sn[FL][2][5];     // face lanes: the neighbours' states
  double gT[FL][2];        //   the ghost temperatures of the lines
  double eh[FL][NP];       //   the diffusive part of the lines' energy sums
  double acc[5][NP];       // line lanes: the other sums of the line's nodes
  {
    const LineArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
    fetch_nodes<N>(A.U, stride, e, tid, u);
    if constexpr (FACE) fetch_faces<N>(A.U, stride, Place(A.mesh, e), e, wtid - 64 * L::LW, sn);
    if (tid < NP) {
      double w = A.basis.inv_w[0];
#pragma unroll
      for (int i = 1; i < NP; ++i) w = tid == i ? A.basis.inv_w[i] : w;
      sW[tid] = w;
    }
  }

  primitives_to_lds<N, VISC>(again(args), sF, again(tid), u);

  do {
    const Place pl(again(args).mesh, e);
    phase_end();

    // ---- line phase: flux differencing; faces on the other wave(s) ---------
    if constexpr (FACE) {
      // per face node: the ghost values of (u, v, w) (halves, line frame; 0..2; that
      // of T stays here), and the face's part of the sums (3..7): -+ half the two-point flux
      // with the ghost and the Lax-Friedrichs dissipation
      // (lambda / 4) (U_own - U_neighbour) (the sums are scaled by 2 at the end)
      const LineArgs& A = again(args);
      const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
      for (int q = 0; q < FL; ++q) {
        const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int l = t.node(h ? N : 0);
          const double ph0 = sF[4 * EB + t.first];
          const double ro = sF[l], un = sF[(1 + t.d) * EB + l], u1 = sF[(1 + t.d1) * EB + l], u2 = sF[(1 + t.d2) * EB + l];
          const double p = sF[4 * EB + l], en = sF[5 * EB + l], T = sF[6 * EB + l];
          const double* s = sn[q][h];
          const double ir = rcp_nr(s[0]);
          double gn = 0.5 * (s[1] * ir), g1 = 0.5 * (s[2] * ir), g2 = 0.5 * (s[3] * ir), gr = 0.5 * s[0];
          double gp = 0.5 * A.ph.gm1 * (s[4] - 4.0 * (gr * (gn * gn + g1 * g1 + g2 * g2)));
          double ge = 0.5 * (s[4] * ir), gt = 2.0 * gp * A.ph.inv_R * ir;
          const bool wall = pl.neighbour(t.d, h) < 0;
          const bool wm = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL;
          const double gR = A.ph.gamma * A.ph.R;
          const double so = fabs(un + un) + sqrt_nr(gR * T), s1 = fabs(gn + gn) + sqrt_nr(gR * gt), r2 = ro + ro;
          const double lam = wall || A.ph.central ? 0.0 : 0.25 * (so >= s1 ? so : s1);
          const double jump[5] = {lam * (r2 - s[0]), lam * (r2 * (un + un) - s[1]), lam * (r2 * (u1 + u1) - s[2]),
                                  lam * (r2 * (u2 + u2) - s[3]), lam * (r2 * (en + en) - s[4])};
          gr = wall ? ro : gr;
          gp = wall ? p : gp;
          ge = wall ? en : ge;
          gn = wall ? -un : gn;
          g1 = wall ? (wm ? u1 : -u1) : g1;
          g2 = wall ? (wm ? u2 : -u2) : g2;
          gT[q][h] = wall ? (wm ? T : 2.0 * A.mesh.T_wall - T) : gt;
          const double rm = ro + gr, m = rm * (un + gn), pm = (p - ph0) + (gp - ph0), sg = h ? 0.5 : -0.5;
          const double o[8] = {gn, g1, g2, sg * m + jump[0], sg * (m * (un + gn) + pm) + jump[1],
                               sg * (m * (u1 + g1)) + jump[2], sg * (m * (u2 + g2)) + jump[3],
                               sg * ((un + gn) * (rm * (en + ge) + (pm + (ph0 + ph0)))) + jump[4]};
#pragma unroll
          for (int k = 0; k < 8; ++k) sF[L::end_at(t.d, 8 * h + k, t.ab)] = o[k];
        }
      }
    } else {
      const LineArgs& A = again(args);
      const LineTask<N> t(again(wtid));
      double q[6][NP];  // rho, velocities in the line frame, p relative to node 0, e (halves)
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        const int l = t.node(m);
        q[0][m] = sF[l];
        q[1][m] = sF[(1 + t.d) * EB + l];
        q[2][m] = sF[(1 + t.d1) * EB + l];
        q[3][m] = sF[(1 + t.d2) * EB + l];
        q[4][m] = sF[4 * EB + l];
        q[5][m] = sF[5 * EB + l];
      }
      // Kennedy-Gruber pairs of half values: with the sums (means) rho, u, v, w,
      // p, e, f = (m, m u + p, m v, m w, u (rho e + p + p0)), m = rho u; p is
      // relative to the line's first node (p0): the multiple of the row sum of Q
      // it leaves out of the momentum vanishes, and so do its rounding errors
      const double ph0 = q[4][0], p0 = ph0 + ph0;
#pragma unroll
      for (int m = 0; m < NP; ++m) q[4][m] -= ph0;
#pragma unroll
      for (int v = 0; v < 5; ++v)
#pragma unroll
        for (int m = 0; m < NP; ++m) acc[v][m] = 0.0;
#pragma unroll
      for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int m = i + 1; m <= N; ++m) {
          const double rho = q[0][i] + q[0][m], un = q[1][i] + q[1][m], pm = q[4][i] + q[4][m];
          const double mass = rho * un;
          const double f[5] = {mass, mass * un + pm, mass * (q[2][i] + q[2][m]), mass * (q[3][i] + q[3][m]),
                               un * (rho * (q[5][i] + q[5][m]) + (pm + p0))};
          const double c = q_im<N>(A.basis, i, m);
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            acc[v][i] += c * f[v];
            acc[v][m] -= c * f[v];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      settle(acc);
    }
    phase_end();

    // ---- line phase: gradients ------------------------------------------------
    double fn[FACE ? FL : 2][3];  // face lanes: (line, end); line lanes: (end, component)
    if constexpr (!FACE) {
      const LineArgs& A = again(args);
      const LineTask<N> t(again(wtid));
      const int nb[2] = {pl.neighbour(t.d, 0), pl.neighbour(t.d, 1)};
      double gh[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int c = 0; c < 3; ++c) gh[h][c] = sF[L::end_at(t.d, 8 * h + c, t.ab)];
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][h ? N : 0] += sF[L::end_at(t.d, 8 * h + 3 + v, t.ab)];
      }
      if (VISC) {
        // the neighbours' normal viscous flux at the ends, in flight over the next phases
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const double* src = A.ffv + static_cast<long long>(nb[h] >= 0 ? nb[h] : e) * (6 * 4 * NF) + (2 * t.d + 1 - h) * (4 * NF);
          // (tangential components at a wall-model wall: the modelled stress)
          const double* tw = src;
          if (nb[h] < 0 && A.mesh.tauw != nullptr && pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL)
            tw = A.mesh.tauw + wall_face_index(A.mesh, pl.ex, pl.ey, pl.ez, t.d, h != 0) * 3 * NF;
          const unsigned ab = t.ab;
          fn[h][0] = load_once(&(src + t.d * NF)[ab]);
          fn[h][1] = load_once(&(tw + t.d1 * NF)[ab]);
          fn[h][2] = load_once(&(tw + t.d2 * NF)[ab]);
        }
        int ad[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) ad[m] = t.node(m);
        double q[NP], g[NP];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int qc = c == 0 ? t.d : (c == 1 ? t.d1 : t.d2);
#pragma unroll
          for (int m = 0; m < NP; ++m) q[m] = sF[(1 + qc) * EB + ad[m]];
          line_derivative<N>(A.basis, q, gh[0][c], gh[1][c], g);
#pragma unroll
          for (int m = 0; m < NP; ++m) sF[(7 + 3 * qc + t.d) * EB + ad[m]] = g[m];
          }
      }
      settle(acc);
    } else if (VISC) {
      // heat flux: it needs the temperature's derivative along the line only
      // (half value; a wall's ghost is 2 q* - q: the own heat flux at an isothermal
      // wall, none at an adiabatic one)
      const LineArgs& A = again(args);
      const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
      for (int q = 0; q < FL; ++q) {
        const LineTask<N> t = face_line<N>(lane, q);
        const int nb[2] = {pl.neighbour(t.d, 0), pl.neighbour(t.d, 1)};
#pragma unroll
        for (int h = 0; h < 2; ++h)
          fn[q][h] = load_once(&(A.ffv + static_cast<long long>(nb[h] >= 0 ? nb[h] : e) * (6 * 4 * NF) +
                                 ((2 * t.d + 1 - h) * 4 + 3) * NF)[static_cast<unsigned>(t.ab)]);
        double T[NP], g[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) T[m] = sF[6 * EB + t.node(m)];
        line_derivative<N>(A.basis, T, gT[q][0], gT[q][1], g);
        const double sk = 0.5 * A.ph.kappa * (t.d == 0 ? pl.sx : (t.d == 1 ? pl.sy : pl.sz));
#pragma unroll
        for (int m = 0; m < NP; ++m) g[m] *= sk * A.basis.inv_w[m];
        if (A.ph.suth)
#pragma unroll
          for (int m = 0; m < NP; ++m) g[m] *= sF[L::MU + t.node(m)];
        const double qw = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL ? -1.0 : 1.0;
        line_derivative<N>(A.basis, g, (nb[0] < 0 ? qw : 0.0) * g[0], (nb[1] < 0 ? qw : 0.0) * g[N], eh[q]);
      }
      settle(eh);
      if (PERSIST) {
        const LineArgs& B = again(args);
        const int en = e + step_e < end_e ? e + step_e : e;
        fetch_faces<N>(B.U, B.mesh.nE * NN, Place(B.mesh, en), en, again(wtid) - 64 * L::LW, sn);
      }
    }
    if (VISC) {
      phase_end();

      // ---- node phase: velocity gradients -> half viscous fluxes (in place) ---
      {
        const LineArgs& A = again(args);
        const int ts = again(tid);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
          const unsigned n = ts + r * BS;
          if (n < NN) {
            const int i = n % NP, j = (n / NP) % NP, k = n / NF;
            const int l = L::at(i, j, k);
            const double c0 = pl.sx * sW[i], c1 = pl.sy * sW[j], c2 = pl.sz * sW[k];
            double mu = A.ph.mu;  // half fluxes: the gradients are those of half velocities
            if (A.ph.suth) mu *= sF[L::MU + l];
            double gr[9];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              gr[3 * c] = c0 * sF[(7 + 3 * c) * EB + l];
              gr[3 * c + 1] = c1 * sF[(8 + 3 * c) * EB + l];
              gr[3 * c + 2] = c2 * sF[(9 + 3 * c) * EB + l];
            }
            const double dd = (2.0 / 3.0) * (gr[0] + gr[4] + gr[8]);
            const double t00 = mu * (gr[0] + gr[0] - dd), t11 = mu * (gr[4] + gr[4] - dd), t22 = mu * (gr[8] + gr[8] - dd);
            const double t01 = mu * (gr[1] + gr[3]), t02 = mu * (gr[2] + gr[6]), t12 = mu * (gr[5] + gr[7]);
            const double uu = 2.0 * sF[EB + l], vv = 2.0 * sF[2 * EB + l], ww = 2.0 * sF[3 * EB + l];
            sF[7 * EB + l] = t00;
            sF[8 * EB + l] = t11;
            sF[9 * EB + l] = t22;
            sF[10 * EB + l] = t01;
            sF[11 * EB + l] = t02;
            sF[12 * EB + l] = t12;
            sF[13 * EB + l] = uu * t00 + vv * t01 + ww * t02;
            sF[14 * EB + l] = uu * t01 + vv * t11 + ww * t12;
            sF[15 * EB + l] = uu * t02 + vv * t12 + ww * t22;
          }
        }
      }
      phase_end();
    }

    // G of this element is in flight over the rest
    __builtin_amdgcn_sched_barrier(0);
    const int tl = again(tid);
    double gA[ROUNDS][5];
    if (RK) {
      const LineArgs& A = again(args);
      const long long stride = A.mesh.nE * NN;
      // (the first stage has no G: it reads U's rows again, mostly from cache)
      const double* G = A.st.read_G ? A.out : A.U;
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
        for (int v = 0; v < 5; ++v)
          gA[r][v] = load_once(&(G + v * stride + static_cast<long long>(e) * NN)[node_of<N>(tl, r)]);
    }

    __builtin_amdgcn_sched_barrier(0);
    // ---- line phase: divergence of the viscous flux --------------------------
    if constexpr (VISC && !FACE) {
      const LineArgs& A = again(args);
      const LineTask<N> t(again(wtid));
      const int nb[2] = {pl.neighbour(t.d, 0), pl.neighbour(t.d, 1)};
      const bool wm = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL;
      int ad[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) ad[m] = t.node(m);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        // tau_qd: the diagonal at 7 + d, (0,1), (0,2), (1,2) at 9 + q + d
        const int qc = c == 1 ? t.d1 : t.d2;
        const int slot = c == 0 ? 7 + t.d : 9 + qc + t.d;
        double f[NP], g[NP], gw[2];
#pragma unroll
        for (int m = 0; m < NP; ++m) f[m] = sF[slot * EB + ad[m]];
        // ghosts: half the neighbour's flux; at a wall 2 f* - f: the own stresses at
        // an isothermal no-slip wall; the own normal stress and the modelled shear
        // stress at a wall-model wall
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool wall = nb[h] < 0;
          const double of_n = !wall ? 0.5 : (wm && c > 0 ? (h ? -1.0 : 1.0) : 0.0);
          const double of_o = !wall ? 0.0 : (wm && c > 0 ? -1.0 : 1.0);
          gw[h] = of_n * fn[h][c] + of_o * f[h ? N : 0];
        }
        line_derivative<N>(A.basis, f, gw[0], gw[1], g);
#pragma unroll
        for (int m = 0; m < NP; ++m) acc[1 + c][m] -= g[m];
      }
      settle(acc);
    } else if constexpr (VISC) {
      // the stresses' work, u . tau_d (a wall's own does no work: ghost -f)
      const LineArgs& A = again(args);
      const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
      for (int q = 0; q < FL; ++q) {
        const LineTask<N> t = face_line<N>(lane, q);
        double f[NP], g[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) f[m] = sF[(13 + t.d) * EB + t.node(m)];
        const double g0 = pl.neighbour(t.d, 0) < 0 ? -f[0] : 0.5 * fn[q][0];
        const double g1 = pl.neighbour(t.d, 1) < 0 ? -f[N] : 0.5 * fn[q][1];
        line_derivative<N>(A.basis, f, g0, g1, g);
#pragma unroll
        for (int m = 0; m < NP; ++m) eh[q][m] += g[m];
      }
      settle(eh);
    }

    __builtin_amdgcn_sched_barrier(0);
    // ---- sums of the three directions, scaling, output -----------------------
    // the next element's first loads are in flight over the exchange (the own
    // state stays in registers for the update: read again here it would mostly
    // come from HBM)
    double un[ROUNDS][5];
    if (PERSIST) {
      const LineArgs& A = again(args);
      const long long stride = A.mesh.nE * NN;
      const int en = e + step_e < end_e ? e + step_e : e;
      fetch_nodes<N>(A.U, stride, en, tl, un);
      if constexpr (FACE && !VISC) fetch_faces<N>(A.U, stride, Place(A.mesh, en), en, again(wtid) - 64 * L::LW, sn);
    }
    phase_end();
    if constexpr (!FACE) {
      const LineTask<N> t(again(wtid));
      double* o = sF + 5 * t.d * EB;
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        const int l = t.node(m);
        o[l] = acc[0][m];
        o[(1 + t.d) * EB + l] = acc[1][m];
        o[(1 + t.d1) * EB + l] = acc[2][m];
        o[(1 + t.d2) * EB + l] = acc[3][m];
        o[4 * EB + l] = acc[4][m];
      }
    } else if constexpr (VISC) {
      const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
      for (int q = 0; q < FL; ++q) {
        const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
        for (int m = 0; m < NP; ++m) sF[(15 + t.d) * EB + t.node(m)] = eh[q][m];
      }
    }
    phase_end();
    double g1[ROUNDS][5], u1[ROUNDS][5];  // Ut or the new G, and the new U
    {
      const LineArgs& A = again(args);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const unsigned n = node_of<N>(tl, r);
        const int i = n % NP, j = (n / NP) % NP, k = n / NF;
        const int l = L::at(i, j, k);
        const double c0 = -2.0 * (pl.sx * sW[i]), c1 = -2.0 * (pl.sy * sW[j]), c2 = -2.0 * (pl.sz * sW[k]);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          double f0 = sF[v * EB + l], f1 = sF[(5 + v) * EB + l], f2 = sF[(10 + v) * EB + l];
          if (VISC && v == 4) {
            f0 -= sF[15 * EB + l];
            f1 -= sF[16 * EB + l];
            f2 -= sF[17 * EB + l];
          }
          const double ut = c0 * f0 + c1 * f1 + c2 * f2;
          if (RK) {
            g1[r][v] = A.st.read_G ? A.st.A * gA[r][v] + A.st.dt * ut : A.st.dt * ut;
            u1[r][v] = u[r][v] + A.st.B * g1[r][v];
          } else {
            g1[r][v] = ut;
          }
        }
      }
    }
    if (PERSIST) {
      // the next element's primitives before this one's stores: a load is waited
      // for together with all stores issued before it
      settle(g1);
      if (RK) settle(u1);
      phase_end();
      primitives_to_lds<N, VISC>(again(args), sF, again(tid), un);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
        for (int v = 0; v < 5; ++v) u[r][v] = un[r][v];
    }
    {
      const LineArgs& A = again(args);
      const long long stride = A.mesh.nE * NN, base = static_cast<long long>(e) * NN;
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const unsigned n = again(tid) + r * BS;
        if (NN % BS == 0 || n < NN)
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            store_once(&(A.out + v * stride + base)[n], g1[r][v]);
            if (RK) store_once(&(A.U_out + v * stride + base)[n], u1[r][v]);
          }
      }
    }
    e += step_e;
  } while (PERSIST && e < end_e);
}

template <int N, bool RK, bool VISC>
__global__ __launch_bounds__(Line<N>::BS) __attribute__((amdgpu_waves_per_eu(N == 7 ? 2 : (N == 5 ? 3 : 4)))) void k_rhs_line(LineArgs) {
  using L = Line<N>;
  constexpr bool PERSIST = N == 7;
  extern __shared__ double lds[];
  const LineArgsPtr args = (LineArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x;
  // elements of this workgroup: those of its XCD (workgroup index modulo 8) in
  // steps of the XCD's workgroups, so that an XCD's workgroups sweep one
  // contiguous range together
  const int blk = static_cast<int>(blockIdx.x);
  int e, step_e = 0, end_e = 0;
  if constexpr (PERSIST) {
    const int nE = static_cast<int>(again(args).mesh.nE), grid = static_cast<int>(gridDim.x), xcd = blk & 7;
    const int q8 = nE >> 3, r8 = nE & 7;
    const int begin = xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8;
    end_e = begin + q8 + (xcd < r8 ? 1 : 0);
    e = begin + (blk >> 3);
    step_e = (grid + 7 - xcd) >> 3;
    if (e >= end_e) return;
  } else {
    e = xcd_remap(blk, gridDim.x);
  }
  // line lane number of this lane (>= LINES: none); face lanes are those of the
  // last FW waves.  At N = 7 which of the four waves that is changes from
  // workgroup to workgroup, so that not all face waves share a SIMD.
  const int turn = PERSIST ? ((blk >> 3) + (blk >> 8)) & 3 : 0;
  const auto line_of = [turn](int t) { return PERSIST ? (t + 64 * turn) & 255 : t; };

  const int wtid = line_of(tid);
  if (__builtin_amdgcn_readfirstlane(wtid) >= 64 * L::LW)
    rhs_line_phases<N, RK, VISC, true>(args, lds, e, step_e, end_e, tid, wtid);
  else
    rhs_line_phases<N, RK, VISC, false>(args, lds, e, step_e, end_e, tid, wtid);
}

template <int N, bool RK>
hipError_t line_n(const LineArgs& a, hipStream_t s) {
  // N = 7: as many workgroups as run at once (two per CU), each fetching its next
  // element while it works on one
  const long long most = N == 7 ? 512 : a.mesh.nE;
  const dim3 grid(static_cast<unsigned>(a.mesh.nE < most ? a.mesh.nE : most)), block(Line<N>::BS);
  const size_t lds = line_lds<N>(a.ph);
  if (a.ph.viscous)
    hipLaunchKernelGGL((k_rhs_line<N, RK, true>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((k_rhs_line<N, RK, false>), grid, block, lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_line(int N, const DevMesh& m, const DevPhys& p, const DevBasis& b, const double* U,
                       const double* ffv, double* out, double* U_out, const Stage& st, bool rk, int* status,
                       hipStream_t s) {
  const LineArgs a{U, ffv, out, U_out, status, m, p, b, st};
  switch (N) {
    case 3: return rk ? line_n<3, true>(a, s) : line_n<3, false>(a, s);
    case 5: return rk ? line_n<5, true>(a, s) : line_n<5, false>(a, s);
    case 7: return rk ? line_n<7, true>(a, s) : line_n<7, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dg
