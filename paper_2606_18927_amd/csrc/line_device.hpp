// Right-hand side (and fused RK stage) with line lanes, for gfx950.
//
// What bounds it (N = 7, 32^3 elements, RK instance, per launch; with one lane per
// node and every node reading its lines from LDS in brackets):
//                       time us        HBM GB   vector instr. 10^6   their issue   LDS busy
//   FP64                799  (986)     3.13     226  (355)           50 %          27 % (55 %)
//   mixed               713  (838)     2.93     279                  69 %          26 % (44 %)
//   entropy-cons. FP64 1069 (1651)     3.13     360  (671)           67 %          22 % (36 %)
//   entropy-cons. mixed 857 (1351)     2.93     403                  91 %          22 %
// (Mixed precision with each direction's parts in one FP32 sum: 662 and 822 us, and a mass
// that a long run loses.)
// A triad moves 3.13 GB in 0.49 ms.  In FP64 a CU holds two workgroups (77 KB LDS, 224
// registers: the whole line and its sums): eight waves have to hide each other's memory,
// LDS and barrier latencies; the entropy-conserving pair is bound by its instructions.
// (Workgroups that loop over elements and fetch the next one early: 4 - 7 % slower; two
// lanes per line: twice as slow, only one workgroup of six waves fits a CU.)
//
// One workgroup works on one element.  Two kinds of phases alternate, with the nodal fields in LDS between them:
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
//
// Mixed precision (R = float): the LDS fields, gradients, viscous fluxes, pair
// fluxes and line sums are FP32; U, G, the primitive recovery, the jumps across
// faces (lifting corrections, Lax-Friedrichs terms as FP64 differences of the two
// sides, the whole Roe flux), the sum of a direction's parts (flux differences, surface
// terms, viscous sums) and over directions, and the RK update stay FP64.
// p, e (entropy-conserving pair: beta, and pi = rho (p - p_ref) / p) and T enter
// relative to the element's first node.  There the faces keep the strong form (own
// end value plus jump), so that no FP32 difference of large values is formed; the
// reference values' part of the energy, e_ref sum D (rho u)# + p_ref sum D u, is
// added back in FP64.
#pragma once

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
  __device__ static constexpr int at(int i, int j, int k) {
    return SWZ ? (i ^ j) + NP * (j ^ k) + NF * k : i + RS * (j + NP * k);
  }
};

// Faces of a line that its face lane takes.  The Roe flux of one face is as long as
// half a line's pairs are together, so with it the line lanes take the upper ones
// themselves where the face waves would be the last: N = 7 has one face wave beside three
// line waves (24^3 step 6.88 ms without, 6.03 with), N = 3 six pairs per line; N = 5 has as
// many face waves as line waves.
template <int N, bool EC>
__host__ __device__ constexpr int line_faces() {
  return EC && N != 5 ? 1 : 2;
}

// LDS fields (of EB values of type R) of a workgroup.  Halves of rho, u, v, w
// (0..3); 4, 5: halves of p and e, entropy-conserving pair beta and |u|^2 / 4; with
// it in mixed precision pi / 2; then T.  From GS on the raw velocity gradients
// GS + 3 q + d, then the half viscous fluxes tau_00, tau_11, tau_22, tau_01, tau_02,
// tau_12, u . tau_d.  The 8 values of each line end (velocity ghosts, face sums) take,
// where a wave holds one direction, gradient fields that this wave alone writes
// after reading them, else a region of their own; mixed precision puts the FP64
// states of the boundary nodes (for the faces) into the gradient fields that are left.
// At the end the directions' sums: FP64 5 d + v (0..14) and their diffusive energy
// parts (15 + d); mixed precision 4 d + (mass, momentum), the energy sums as FP64
// (12 + 2 d), the diffusive parts (18 + d), the surface terms and the viscous sums apart.
// Behind the fields: the line ends' ghost temperatures, mu(T) / mu (Sutherland's law only).
template <int N, typename R, bool EC>
struct Fields {
  using L = Line<N>;
  static constexpr bool MIXED = sizeof(R) == 4;
  static constexpr int TS = EC && MIXED ? 7 : 6, GS = TS + 1;
  // Mixed precision sums in FP32 and adds the sums in FP64: a direction's flux differences,
  // its surface terms and, with the Kennedy-Gruber pair, its viscous sums (VS + 3 d + c).
  // At N = 5 and 7 these nine fields would cost a CU a workgroup and follow in a second round
  // (N = 5, 24^3: 1015 us a step with 30 fields, 985 so; all in one FP32 sum 945, with
  // the rounding error of the larger parts in the smaller ones).
  static constexpr bool SPLIT = MIXED && !EC, TWICE = SPLIT && N != 3;
  static constexpr int VS = TWICE ? 0 : 21;
  static constexpr int COUNT = !MIXED ? 18 : (SPLIT && !TWICE ? 30 : 21);
  static constexpr int ENDS = COUNT * L::EB;
  static constexpr int GT = ENDS + (L::UNIFORM ? 0 : 16 * L::LINES);
  // (where the lane that forms them also reads them back, in registers: at N = 5 three
  // workgroups with Sutherland's law fit a CU without the ghost temperatures in LDS)
  static constexpr bool KEEP_T = !L::UNIFORM && line_faces<N, EC>() == 2;
  static constexpr int MU = GT + (KEEP_T ? 0 : 2 * L::LINES);
  static constexpr int OWN = (L::UNIFORM ? GS + 6 : GS) * L::EB;  // 5 FP64 values per boundary node
  static constexpr int NB = n_face_nodes<N>();
  static_assert(!MIXED || OWN + 10 * NB <= (L::UNIFORM ? COUNT : GS + 9) * L::EB, "boundary states fit");
  static constexpr int HEAD = 16;  // FP64 values before the fields: 1 / w_i, and the reference values
  __device__ static int end_at(int d, int k, int ab) {
    return L::UNIFORM ? (GS + 3 * (k >> 3) + d) * L::EB + (k & 7) * L::NF + ab : ENDS + k * L::LINES + d * L::NF + ab;
  }
  // component v of the surface term at end h of a line, in mixed precision at the end: where
  // the faces put it, or behind the sums (over the ghost temperatures and mu(T) / mu)
  __device__ static int surface_at(int d, int h, int v, int ab) {
    return L::UNIFORM ? COUNT * L::EB + (5 * h + v) * L::LINES + d * L::NF + ab : end_at(d, 8 * h + 3 + v, ab);
  }
  static size_t bytes(const DevPhys& p) {
    const size_t used = static_cast<size_t>(MU) + (p.viscous && p.suth ? L::EB : 0);
    const size_t sums = MIXED && L::UNIFORM ? static_cast<size_t>(COUNT) * L::EB + 10 * L::LINES : 0;
    return HEAD * sizeof(double) + sizeof(R) * (used > sums ? used : sums);
  }
};

// Arguments of the kernel.  The kernel reads them from the kernel-argument
// segment where a phase needs them, instead of holding all of them (the
// coefficients among them) in scalar registers from the start.
struct LineArgs {
  const double* U;
  const void* ffv;  // R*
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
template <int N, typename R>
__device__ inline R q_im(const DevBasis& b, int i, int m) {
  const int a = i + m > N ? N - m : i, c = i + m > N ? N - i : m;
  const int id = a * N - a * (a - 1) + c - a - 1;
  if constexpr (sizeof(R) == 4)
    return b.Qf[id];
  else
    return b.Q[id];
}

// The s-th of the n pairs at one distance, by its lower node: from the line's two ends
// inwards.  All sums over pairs run from the farthest pairs (small Q) to the nearest, and
// the end values come last: the partial sums stay small, and the rounding of row N - i
// mirrors that of row i.  (Row by row from node 0, constant flow plus noise in FP32:
// twice the rounding error in the first rows, and a mean error of the line's sum of 3e-10
// of the flux, now below 5e-11, which a long run accumulates as a loss of mass.)
__device__ constexpr int pair_low(int n, int s) { return s & 1 ? n - 1 - (s >> 1) : s >> 1; }

// g_i = sum_{m != i} Q_im q_m plus the two ghost values; with STRONG the ghost
// values are the jumps to them from the own end values.
template <int N, typename R, bool STRONG>
__device__ inline void line_derivative(const DevBasis& b, const R (&q)[N + 1], R ghost_lo, R ghost_hi, R (&g)[N + 1]) {
#pragma unroll
  for (int i = 0; i <= N; ++i) g[i] = R(0);
#pragma unroll
  for (int dist = N; dist > 0; --dist)
#pragma unroll
    for (int s = 0; s <= N - dist; ++s) {
      const int i = pair_low(N + 1 - dist, s), m = i + dist;
      const R c = q_im<N, R>(b, i, m);
      g[i] += c * q[m];
      g[m] -= c * q[i];
    }
  if (STRONG) {
    g[0] -= R(0.5) * q[0];
    g[N] += R(0.5) * q[N];
  }
  g[0] -= R(0.5) * ghost_lo;
  g[N] += R(0.5) * ghost_hi;
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
  // (scales: none on curved elements)
  __device__ Place(const DevMesh& m, int e, bool scales = true) {
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
    sx = scales ? ((Table)(uintptr_t)m.s[0])[ex] : 0.0;
    sy = scales ? ((Table)(uintptr_t)m.s[1])[ey] : 0.0;
    sz = scales ? ((Table)(uintptr_t)m.s[2])[ez] : 0.0;
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

// The neighbour's state at end h of line t, in the line frame (rho, momentum along
// the line and across, E).
template <int N>
__device__ inline void fetch_end(const double* __restrict__ U, long long stride, const Place& pl, int e,
                                 const LineTask<N>& t, int h, double (&s)[5]) {
  const int nb = pl.neighbour(t.d, h);
  const unsigned o = t.end_node(h ? 0 : N);
  const double* p = U + static_cast<long long>(nb >= 0 ? nb : e) * Line<N>::NN;
  s[0] = p[o];
  s[1] = (p + (1 + t.d) * stride)[o];
  s[2] = (p + (1 + t.d1) * stride)[o];
  s[3] = (p + (1 + t.d2) * stride)[o];
  s[4] = (p + 4 * stride)[o];
}

template <int N>
__device__ inline void fetch_faces(const double* __restrict__ U, long long stride, const Place& pl, int e, int lane,
                                   double (&sn)[Line<N>::FL][2][5]) {
#pragma unroll
  for (int q = 0; q < Line<N>::FL; ++q) {
    const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
    for (int h = 0; h < 2; ++h) fetch_end<N>(U, stride, pl, e, t, h, sn[q][h]);
  }
}

// Values that have to exist at this point: the compiler would else sink the sums
// that make them into a later phase, and hold all their operands until then.
template <typename R, int A, int B>
__device__ __forceinline__ void settle(R (&x)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) asm volatile("" : "+v"(x[a][b]));
}

// Waves per SIMD the registers are bounded for: what LDS lets a CU hold (N = 7: 77 KB
// in FP64, 45 KB mixed), or what the entropy-conserving pair needs without spilling
// more than a few values (N = 5 in FP64 spills 44 at one wave more: smooth states
// 3.38 -> 3.10 ms a step at 32^3, rough ones, with spills inside the loop over pairs,
// 9.08 -> 13.63).  With that pair N = 3 in FP64 takes three waves and 10 spilled values
// before two and none (48^3: 6.25 -> 5.14 ms a step; rough 8.81 -> 7.92), N = 5 mixed
// four, which its registers just fit (32^3: 3.30 -> 3.13 ms; rough 6.11 -> 5.44).
template <int N, typename R, bool EC>
__host__ __device__ constexpr int line_waves() {
  return sizeof(R) == 8 ? (N == 7 ? 2 : (N == 5 ? (EC ? 2 : 3) : (EC ? 3 : 4))) : (N == 7 ? 3 : 4);
}

// A phase boundary: a workgroup barrier that no instruction is scheduled across
// (the phases' values would else overlap and spill).
__device__ __forceinline__ void phase_end() {
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
}

// After this lanes of a wave overwrite in LDS what other lanes of it read before.  The
// hardware keeps a wave's LDS accesses in order, this the compiler, which could prove a lane's
// own accesses apart; it costs no instruction.
__device__ __forceinline__ void wave_reuse() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Node phase: primitives of the states u into the LDS fields (mixed precision:
// relative to the state s0 of the element's first node, and the boundary nodes' own
// states).
template <int N, typename R, bool VISC, bool EC>
__device__ __forceinline__ void primitives_to_lds(const LineArgs& A, double* const head, R* const sF, const int tid,
                                                 const double (&u)[Line<N>::ROUNDS][5], const double (&s0)[5]) {
  using L = Line<N>;
  using Fd = Fields<N, R, EC>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, ROUNDS = L::ROUNDS;
  constexpr bool MIXED = Fd::MIXED;
  double p_ref = 0.0, e_ref = 0.0, T_ref = 0.0, beta_ref = 0.0;
  if (MIXED && A.ph.mixed_ref) {
    const Prim P = primitives(s0, A.ph);
    p_ref = P.p;
    // (entropy-conserving pair: the internal energy p / ((gamma - 1) rho))
    e_ref = EC ? P.p / (A.ph.gm1 * P.rho) : P.e;
    T_ref = P.T;
    beta_ref = 0.5 * P.rho / P.p;
  }
  if (MIXED && tid == 0) {
    head[NP] = p_ref;
    head[NP + 1] = e_ref;
    head[NP + 2] = beta_ref;
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const unsigned n = tid + r * L::BS;
    if (n < NN) {
      const double* s = u[r];
      const double ir = rcp_nr(s[0]);
      const double vx = s[1] * ir, vy = s[2] * ir, vz = s[3] * ir;
      const double q2 = vx * vx + vy * vy + vz * vz;
      const double p = A.ph.gm1 * (s[4] - 0.5 * s[0] * q2);
      const double T = p * A.ph.inv_R * ir;
      if (!(s[0] > 0.0) || !(p > 0.0)) A.status[0] = 1;
      const int i = n % NP, j = (n / NP) % NP, k = n / NF;
      const int l = L::at(i, j, k);
      sF[l] = static_cast<R>(0.5 * s[0]);
      sF[EB + l] = static_cast<R>(0.5 * vx);
      sF[2 * EB + l] = static_cast<R>(0.5 * vy);
      sF[3 * EB + l] = static_cast<R>(0.5 * vz);
      if (EC) {
        const double ip = rcp_nr(p);
        sF[4 * EB + l] = static_cast<R>((MIXED ? 0.5 * s[0] * ip : quot(0.5 * s[0], p, ip)) - beta_ref);
        sF[5 * EB + l] = static_cast<R>(0.25 * q2);
        if (MIXED) sF[6 * EB + l] = static_cast<R>(0.5 * (s[0] * (p - p_ref) * ip));
      } else {
        sF[4 * EB + l] = static_cast<R>(0.5 * (p - p_ref));
        sF[5 * EB + l] = static_cast<R>(0.5 * (s[4] * ir - e_ref));
      }
      sF[Fd::TS * EB + l] = static_cast<R>(T - T_ref);
      if (VISC && A.ph.suth) sF[Fd::MU + l] = static_cast<R>(viscosity_ratio(A.ph, T));
      if (MIXED && (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N)) {
        double* own = reinterpret_cast<double*>(sF + Fd::OWN) + face_node_index<N>(i, j, k);
#pragma unroll
        for (int v = 0; v < 5; ++v) own[v * Fd::NB] = s[v];
      }
    }
  }
}

// Roe's dissipation sum_k |lambda_k| alpha_k r_k across a face, in the line frame
// (L = lower side, R = upper side; primitives (rho, u along the line, v, w, p) and
// total energies E), linearised at the Roe average: sqrt(rho)-weighted u and
// H = (E + p) / rho, rho~ = sqrt(rho_L rho_R), a~^2 = (gamma - 1)(H~ - |u~|^2 / 2).
// Waves: acoustic u~ -+ a~, alpha = ([[p]] -+ rho~ a~ [[u]]) / (2 a~^2),
// r = (1, u~ -+ a~, v~, w~, H~ -+ u~ a~) with Harten-Hyman |lambda|; entropy u~,
// alpha = [[rho]] - [[p]] / a~^2, r = (1, u~, v~, w~, |u~|^2 / 2); shear u~ with
// rho~ (0, 0, [[v]], [[w]], v~ [[v]] + w~ [[w]]).
__device__ inline void roe_line(const double (&Lp)[5], double EL, const double (&Rp)[5], double ER, double gamma,
                                double (&D)[5]) {
  const double sl = sqrt_nr(Lp[0]), sr = sqrt_nr(Rp[0]);
  const double isum = rcp_nr(sl + sr);
  const double wl = sl * isum, wr = sr * isum;
  const double iL = rcp_nr(Lp[0]), iR = rcp_nr(Rp[0]);
  const double u = wl * Lp[1] + wr * Rp[1], v = wl * Lp[2] + wr * Rp[2], w = wl * Lp[3] + wr * Rp[3];
  const double H = quot(wl * (EL + Lp[4]), Lp[0], iL) + quot(wr * (ER + Rp[4]), Rp[0], iR);
  const double q2 = u * u + v * v + w * w;
  const double a2 = (gamma - 1.0) * (H - 0.5 * q2);
  const double a = sqrt_nr(a2), ia2 = rcp_nr(a2);
  const double rho = sl * sr;
  const double dp = Rp[4] - Lp[4], du = Rp[1] - Lp[1], dv = Rp[2] - Lp[2], dw = Rp[3] - Lp[3];
  const double al1 = 0.5 * quot(dp - rho * a * du, a2, ia2);
  const double al5 = 0.5 * quot(dp + rho * a * du, a2, ia2);
  const double al2 = (Rp[0] - Lp[0]) - quot(dp, a2, ia2);
  const double cl = sqrt_nr(quot(gamma * Lp[4], Lp[0], iL)), cr = sqrt_nr(quot(gamma * Rp[4], Rp[0], iR));
  const double l1 = hh_abs(u - a, Lp[1] - cl, Rp[1] - cr);
  const double l5 = hh_abs(u + a, Lp[1] + cl, Rp[1] + cr);
  const double l2 = fabs(u);
  const double t1 = l1 * al1, t5 = l5 * al5, t2 = l2 * al2, ts = l2 * rho, t = t1 + t2 + t5;
  D[0] = t;
  D[1] = t * u + (t5 - t1) * a;
  D[2] = t * v + ts * dv;
  D[3] = t * w + ts * dw;
  D[4] = t1 * (H - u * a) + t2 * (0.5 * q2) + t5 * (H + u * a) + ts * (v * dv + w * dw);
}

// F = atanh f / f and G = 1 / F for u = f^2 below 1e-2 (dropped terms below 1e-17).
__device__ inline void ln_series(double u, double& F, double& G) {
  F = 1.0 + u * (1.0 / 3.0 + u * (1.0 / 5.0 + u * (1.0 / 7.0 + u * (1.0 / 9.0 + u * (1.0 / 11.0 + u * (1.0 / 13.0 + u * (1.0 / 15.0)))))));
  G = rcp_nr(F);
}

// Chandrashekar's flux of two states (rho, u along the line, v, w) with
// beta = rho / (2 p) and |u|^2 = q2, pressure relative to pl in the momentum.  LONG: the
// logarithmic means by their long series, else chosen (ec_means).
template <bool LONG = false>
__device__ inline void ec_pair(const double (&a)[4], double ba, double qa, const double (&b)[4], double bb, double qb,
                               double gm1, double pl, double (&f)[5]) {
  double rho_ln, inv_beta_ln, p_hat;
  if constexpr (LONG) {
    const double sr = a[0] + b[0], sb = ba + bb, x = rcp_nr(sr * sb);
    const double ir = sb * x, ib = sr * x, fr = (a[0] - b[0]) * ir, fb = (ba - bb) * ib;
    double F, G, unused;
    ln_series(fr * fr, unused, G);
    ln_series(fb * fb, F, unused);
    rho_ln = 0.5 * sr * G;
    inv_beta_ln = 2.0 * ib * F;
    p_hat = 0.5 * sr * ib;
  } else {
    ec_means(a[0], b[0], ba, bb, rho_ln, inv_beta_ln, p_hat);
  }
  const double u = 0.5 * (a[1] + b[1]), v = 0.5 * (a[2] + b[2]), w = 0.5 * (a[3] + b[3]);
  f[0] = rho_ln * u;
  f[1] = f[0] * u + (p_hat - pl);
  f[2] = f[0] * v;
  f[3] = f[0] * w;
  f[4] = f[0] * (0.5 / gm1 * inv_beta_ln - 0.25 * (qa + qb) + (u * u + v * v + w * w)) + p_hat * u;
}

// The same in FP32 relative to (beta_ref, p_ref) of the element (mixed precision),
// of half values a, b = (rho, u, v, w) / 2, beta - beta_ref, |u|^2 / 4, pi / 2 with
// pi = rho (p - p_ref) / p: with sb = beta_a + beta_b,
//   p^ - p_ref = (pi_a + pi_b) / (2 sb),
//   1 / beta_ln - 1 / beta_ref = (2 (F - 1) - (dbeta_a + dbeta_b) / beta_ref) / sb,
// F = atanh f / f of the beta pair, so no FP32 difference of O(p_ref) terms is formed;
// f = f#_EC - (0, p_ref, 0, 0, F_rho e_ref + p_ref {{u}}).  SERIES: both logarithmic
// means by their series (f^2 below 1e-2, dropped terms below 1.1e-9 in F, 3e-10 in G, where
// an FP32 rounding of the means is 6e-8).
template <bool SERIES>
__device__ inline void ec_pair_ref(const float* a, const float* b, float kap, float beta_ref, float ibr, float (&f)[5]) {
  const float sr = a[0] + b[0], sdb = a[4] + b[4];
  const float sb = 2.0f * beta_ref + sdb;
  const float x = __builtin_amdgcn_rcpf(sr * sb);
  const float ir = sb * x, ib = sr * x;
  const float fr = (a[0] - b[0]) * ir, fb = (a[4] - b[4]) * ib;
  const float ur = fr * fr, ub = fb * fb;
  float G = 1.0f - ur * (1.0f / 3.0f + ur * (4.0f / 45.0f + ur * (44.0f / 945.0f)));
  float Fs = ub * (1.0f / 3.0f + ub * (0.2f + ub * (1.0f / 7.0f)));
  if (!SERIES) {
    if (ur >= 1e-2f) G = fr / atanhf(fr);
    if (ub >= 1e-2f) Fs = atanhf(fb) / fb - 1.0f;
  }
  const float u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3];
  const float m = sr * G * u;
  const float dp = (a[6] + b[6]) * ib;
  const float dib = (2.0f * Fs - sdb * ibr) * ib;
  f[0] = m;
  f[1] = m * u + dp;
  f[2] = m * v;
  f[3] = m * w;
  f[4] = m * (kap * dib - (a[5] + b[5]) + (u * u + v * v + w * w)) + dp * u;
}

// What one face node adds to its line's sums.  FP64: the ghost velocities (halves)
// gv and temperature gT, and -+ half the surface flux (its central part the pair flux
// with the ghost) in fs.  Mixed precision: the jumps to the ghosts, and -+ half
// (surface flux - own flux).  so, sn: own and neighbour's state in the line frame
// (FP64: so only in mixed precision, else o = own fields and pl = the line's p0).
template <int N, typename R, bool EC>
__device__ __forceinline__ void face_values(const LineArgs& A, const R* sF, const LineTask<N>& t, int h, bool wall,
                                            const double (&sn)[5], R (&gv)[3], R& gT, R (&fs)[5]) {
  using L = Line<N>;
  using Fd = Fields<N, R, EC>;
  constexpr int EB = L::EB;
  const bool wm = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL;
  const double irn = rcp_nr(sn[0]);
  const double vn[3] = {sn[1] * irn, sn[2] * irn, sn[3] * irn};
  const double q2n = vn[0] * vn[0] + vn[1] * vn[1] + vn[2] * vn[2];
  const double pn = A.ph.gm1 * (sn[4] - 0.5 * sn[0] * q2n);
  const double Tn = pn * A.ph.inv_R * irn;
  if constexpr (!Fd::MIXED) {
    const int l = t.node(h ? N : 0);
    const double ro = sF[l];
    const double vo[3] = {sF[(1 + t.d) * EB + l], sF[(1 + t.d1) * EB + l], sF[(1 + t.d2) * EB + l]};
    const double f4 = sF[4 * EB + l], f5 = sF[5 * EB + l], T = sF[Fd::TS * EB + l];
    gv[0] = wall ? -vo[0] : 0.5 * vn[0];
    gv[1] = wall ? (wm ? vo[1] : -vo[1]) : 0.5 * vn[1];
    gv[2] = wall ? (wm ? vo[2] : -vo[2]) : 0.5 * vn[2];
    gT = wall ? (wm ? T : 2.0 * A.mesh.T_wall - T) : Tn;
    const double sg = h ? 0.5 : -0.5;
    if constexpr (EC) {
      const double pl = sF[t.first] * rcp_nr(sF[4 * EB + t.first]);
      const double po = quot(ro, f4, rcp_nr(f4)), r2 = ro + ro, q2o = 4.0 * f5;
      const double a[4] = {r2, vo[0] + vo[0], vo[1] + vo[1], vo[2] + vo[2]};
      const double bn = quot(0.5 * sn[0], pn, rcp_nr(pn));
      const double b[4] = {wall ? r2 : sn[0], gv[0] + gv[0], gv[1] + gv[1], gv[2] + gv[2]};
      double f[5];
      ec_pair(a, f4, q2o, b, wall ? f4 : bn, wall ? q2o : q2n, A.ph.gm1, pl, f);
      double D[5] = {0, 0, 0, 0, 0};
      if (!A.ph.central) {
        const double Po[5] = {a[0], a[1], a[2], a[3], po}, Pn[5] = {sn[0], vn[0], vn[1], vn[2], pn};
        const double Eo = po / A.ph.gm1 + ro * q2o;
        double X[5], Y[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          X[v] = h ? Po[v] : Pn[v];
          Y[v] = h ? Pn[v] : Po[v];
        }
        roe_line(X, h ? Eo : sn[4], Y, h ? sn[4] : Eo, A.ph.gamma, D);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) fs[v] = sg * (wall ? f[v] : f[v] - 0.5 * D[v]);
    } else {
      const double ph0 = sF[4 * EB + t.first];
      const double r2 = ro + ro, g2 = A.ph.gamma * (f4 + f4), gn = A.ph.gamma * pn;
      const double so = fabs(vo[0] + vo[0]) + sqrt_edge(quot(g2, r2, rcp_nr(r2))), s1 = fabs(vn[0]) + sqrt_edge(quot(gn, sn[0], irn));
      const double lam = wall || A.ph.central ? 0.0 : 0.25 * (so >= s1 ? so : s1);
      const double rm = ro + (wall ? ro : 0.5 * sn[0]), un = vo[0] + gv[0], m = rm * un;
      const double pm = (f4 - ph0) + ((wall ? f4 : 0.5 * pn) - ph0), em = f5 + (wall ? f5 : 0.5 * (sn[4] * irn));
      fs[0] = sg * m + lam * (r2 - sn[0]);
      fs[1] = sg * (m * un + pm) + lam * (r2 * (vo[0] + vo[0]) - sn[1]);
      fs[2] = sg * (m * (vo[1] + gv[1])) + lam * (r2 * (vo[1] + vo[1]) - sn[2]);
      fs[3] = sg * (m * (vo[2] + gv[2])) + lam * (r2 * (vo[2] + vo[2]) - sn[3]);
      fs[4] = sg * (un * (rm * em + (pm + (ph0 + ph0)))) + lam * (r2 * (f5 + f5) - sn[4]);
    }
  } else {
    const unsigned a = static_cast<unsigned>(t.ab) % L::NP, b = static_cast<unsigned>(t.ab) / L::NP;
    const int n = h ? N : 0;
    const double* own = reinterpret_cast<const double*>(sF + Fd::OWN) +
                        face_node_index<N>(t.d == 0 ? n : a, t.d == 0 ? a : (t.d == 1 ? n : b), t.d == 2 ? n : b);
    const double so[5] = {own[0], own[(1 + t.d) * Fd::NB], own[(1 + t.d1) * Fd::NB], own[(1 + t.d2) * Fd::NB],
                          own[4 * Fd::NB]};
    const double iro = rcp_nr(so[0]);
    const double vo[3] = {so[1] * iro, so[2] * iro, so[3] * iro};
    const double q2o = vo[0] * vo[0] + vo[1] * vo[1] + vo[2] * vo[2];
    const double po = A.ph.gm1 * (so[4] - 0.5 * so[0] * q2o);
    const double To = po * A.ph.inv_R * iro;
    gv[0] = static_cast<R>(wall ? -vo[0] : 0.5 * (vn[0] - vo[0]));
    gv[1] = static_cast<R>(wall ? (wm ? 0.0 : -vo[1]) : 0.5 * (vn[1] - vo[1]));
    gv[2] = static_cast<R>(wall ? (wm ? 0.0 : -vo[2]) : 0.5 * (vn[2] - vo[2]));
    gT = static_cast<R>(wall ? (wm ? 0.0 : 2.0 * (A.mesh.T_wall - To)) : Tn - To);
    const R sg = h ? R(0.5) : R(-0.5);
    if constexpr (EC) {
      const double fo[5] = {so[1], so[1] * vo[0] + po, so[1] * vo[1], so[1] * vo[2], (so[4] + po) * vo[0]};
      const double a4[4] = {so[0], vo[0], vo[1], vo[2]}, b4[4] = {sn[0], vn[0], vn[1], vn[2]};
      double f[5], D[5] = {0, 0, 0, 0, 0};
      ec_pair(a4, quot(0.5 * so[0], po, rcp_nr(po)), q2o, b4, quot(0.5 * sn[0], pn, rcp_nr(pn)), q2n, A.ph.gm1, 0.0, f);
      if (!A.ph.central) {
        const double Po[5] = {so[0], vo[0], vo[1], vo[2], po}, Pn[5] = {sn[0], vn[0], vn[1], vn[2], pn};
        double X[5], Y[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          X[v] = h ? Po[v] : Pn[v];
          Y[v] = h ? Pn[v] : Po[v];
        }
        roe_line(X, h ? so[4] : sn[4], Y, h ? sn[4] : so[4], A.ph.gamma, D);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double F = wall ? (v == 1 ? po : 0.0) : f[v] - 0.5 * D[v];
        fs[v] = sg * static_cast<R>(F - fo[v]);
      }
    } else {
      // in the differences dx = x_n - x_o, formed in FP64 and rounded once; with
      // m_o = rho_o u_o and dm = {{rho}}{{u}} - m_o = (drho / 2) u_o + {{rho}} (du / 2):
      // f# - f(own) = (dm, dm {{u_a}} + m_o du_a / 2 (+ dp / 2 along the line),
      //                dm {{e}} + m_o de / 2 + {{u}} dp / 2 + p_o du / 2)
      const float uo[3] = {static_cast<float>(vo[0]), static_cast<float>(vo[1]), static_cast<float>(vo[2])};
      const float ro = static_cast<float>(so[0]), po32 = static_cast<float>(po), mo = ro * uo[0];
      const float hdr = 0.5f * static_cast<float>(sn[0] - so[0]);
      const float hdu[3] = {0.5f * static_cast<float>(vn[0] - vo[0]), 0.5f * static_cast<float>(vn[1] - vo[1]),
                            0.5f * static_cast<float>(vn[2] - vo[2])};
      const float hdp = 0.5f * static_cast<float>(pn - po);
      const double eo = so[4] * iro;
      const float hde = 0.5f * static_cast<float>(sn[4] * irn - eo);
      const float um = uo[0] + hdu[0];
      const float dm = hdr * uo[0] + (ro + hdr) * hdu[0];
      float c[5] = {dm, dm * um + mo * hdu[0] + hdp, dm * (uo[1] + hdu[1]) + mo * hdu[1],
                    dm * (uo[2] + hdu[2]) + mo * hdu[2],
                    dm * (static_cast<float>(eo) + hde) + mo * hde + um * hdp + po32 * hdu[0]};
      if (!A.ph.central) {
        const float gR = static_cast<float>(A.ph.gamma * A.ph.R);
        const float co = fabsf(uo[0]) + sqrtf(gR * static_cast<float>(To));
        const float cn = fabsf(static_cast<float>(vn[0])) + sqrtf(gR * static_cast<float>(Tn));
        const float sl = (h ? -0.5f : 0.5f) * (co >= cn ? co : cn);
#pragma unroll
        for (int v = 0; v < 5; ++v) c[v] += sl * static_cast<float>(sn[v] - so[v]);
      }
      const float cw[5] = {-mo, -mo * uo[0], -mo * uo[1], -mo * uo[2], -static_cast<float>(so[4] + po) * uo[0]};
#pragma unroll
      for (int v = 0; v < 5; ++v) fs[v] = sg * (wall ? cw[v] : c[v]);
    }
  }
}

// The pair sums acc[v][i] = sum_{m != i} Q_im f#_v(i, m) of a line with the
// entropy-conserving pair for states with larger jumps.  LONG: the logarithmic means by
// their long series; else they choose between series and atanh pair by pair.  Not
// unrolled (a second unrolled version spills registers into the usual one): the sums
// of row m are selected by factors 0 and 1.
template <int N, typename R, bool LONG>
__device__ inline void ec_rows(const LineArgs& A, const R* sF, const double* head, const LineTask<N>& t, double pl,
                               R (&acc)[5][N + 1]) {
  using L = Line<N>;
  constexpr int NP = N + 1, EB = L::EB, NFLD = sizeof(R) == 4 ? 7 : 6;
  const float br = static_cast<float>(head[NP + 2]), ibr = static_cast<float>(1.0 / head[NP + 2]);
#pragma unroll 1
  for (int i = 0; i < N; ++i) {
    R a[NFLD], s[5] = {0, 0, 0, 0, 0};
    const auto load = [&](int m, R* x) {
      const int l = t.node(m);
      x[0] = sF[l];
      x[1] = sF[(1 + t.d) * EB + l];
      x[2] = sF[(1 + t.d1) * EB + l];
      x[3] = sF[(1 + t.d2) * EB + l];
      x[4] = sF[4 * EB + l];
      x[5] = sF[5 * EB + l];
      if constexpr (NFLD == 7) x[6] = sF[6 * EB + l];
    };
    load(i, a);
#pragma unroll 1
    for (int m = N; m > i; --m) {
      R b[NFLD], f[5];
      load(m, b);
      if constexpr (NFLD == 7) {
        ec_pair_ref<false>(a, b, static_cast<float>(0.5 / A.ph.gm1), br, ibr, f);
      } else {
        const double x[4] = {a[0] + a[0], a[1] + a[1], a[2] + a[2], a[3] + a[3]};
        const double y[4] = {b[0] + b[0], b[1] + b[1], b[2] + b[2], b[3] + b[3]};
        ec_pair<LONG>(x, a[4], 4.0 * a[5], y, b[4], 4.0 * b[5], A.ph.gm1, pl, f);
      }
      const R c = q_im<N, R>(A.basis, i, m);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        f[v] *= c;
        s[v] += f[v];
      }
#pragma unroll
      for (int r = 1; r < NP; ++r) {
        const R sel = r == m ? R(-1) : R(0);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][r] += sel * f[v];
      }
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const R sel = r == i ? R(1) : R(0);
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[v][r] += sel * s[v];
    }
  }
}

// The phases of a workgroup as its face waves (FACE) or line waves run them: the two
// run the same node phases and meet at the same barriers.  tid: the lane's number
// in the node phases; wtid: its line (>= 64 LW: face lane).
template <int N, typename R, bool RK, bool VISC, bool EC, bool FACE>
__device__ __forceinline__ void rhs_line_phases(const LineArgsPtr args, double* const head, const int e, const int tid,
                                               const int wtid) {
  using L = Line<N>;
  using Fd = Fields<N, R, EC>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, BS = L::BS, ROUNDS = L::ROUNDS, FL = L::FL;
  constexpr int GS = Fd::GS;
  constexpr bool MIXED = Fd::MIXED;
  double* const sW = head;
  R* const sF = reinterpret_cast<R*>(head + Fd::HEAD);
  double u[ROUNDS][5];
  double sn[FL][2][5];     // face lanes, Kennedy-Gruber pair: the neighbours' states
  R eh[FL][NP];            // face lanes: the diffusive part of the lines' energy sums
  R acc[5][NP];            // line lanes: the other sums of the line's nodes
  constexpr int HF = line_faces<N, EC>();
  double su[EC ? 2 : 1][5];  // entropy-conserving pair: neighbours' states, a line lane's upper, a face lane's first line's
  const auto fetch_su = [&](const LineArgs& A, int e) {
    if constexpr (FACE && EC)
#pragma unroll
      for (int h = 0; h < HF; ++h)
        fetch_end<N>(A.U, A.mesh.nE * NN, Place(A.mesh, e), e, face_line<N>(again(wtid) - 64 * L::LW, 0), h, su[h]);
    if constexpr (!FACE && HF == 1)
      fetch_end<N>(A.U, A.mesh.nE * NN, Place(A.mesh, e), e, LineTask<N>(again(wtid)), 1, su[0]);
  };
  {
    const LineArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
    fetch_nodes<N>(A.U, stride, e, tid, u);
    double s0[5] = {1, 0, 0, 0, 1};
    if constexpr (MIXED) {  // (scalar loads: U is constant while the kernel runs)
      typedef const __attribute__((address_space(4))) double* Row;
#pragma unroll
      for (int v = 0; v < 5; ++v) s0[v] = *(Row)(uintptr_t)(A.U + v * stride + static_cast<long long>(e) * NN);
    }
    if constexpr (FACE && !EC) fetch_faces<N>(A.U, stride, Place(A.mesh, e), e, wtid - 64 * L::LW, sn);
    fetch_su(A, e);
    if (tid < NP) {
      double w = A.basis.inv_w[0];
#pragma unroll
      for (int i = 1; i < NP; ++i) w = tid == i ? A.basis.inv_w[i] : w;
      sW[tid] = w;
    }
    primitives_to_lds<N, R, VISC, EC>(again(args), head, sF, again(tid), u, s0);
  }

  const Place pl(again(args).mesh, e);
  phase_end();

  // ---- line phase: flux differencing; faces (on the other wave(s)) ---------
  R gt[2];  // ghost temperatures
  const auto face = [&](const LineTask<N>& t, int h, const double (&s)[5]) {
    R gv[3], gT, fs[5];
    face_values<N, R, EC>(again(args), sF, t, h, pl.neighbour(t.d, h) < 0, s, gv, gT, fs);
#pragma unroll
    for (int k = 0; k < 3; ++k) sF[Fd::end_at(t.d, 8 * h + k, t.ab)] = gv[k];
#pragma unroll
    for (int k = 0; k < 5; ++k) sF[Fd::end_at(t.d, 8 * h + 3 + k, t.ab)] = fs[k];
    if constexpr (Fd::KEEP_T)
      gt[h] = gT;
    else
      sF[Fd::GT + h * L::LINES + t.d * NF + t.ab] = gT;
  };
  if constexpr (FACE) {
    const LineArgs& A = again(args);
    const int lane = again(wtid) - 64 * L::LW;
    if constexpr (EC) {
      // one line after the other (the Roe flux is long), the next one's states in
      // flight meanwhile
      const long long stride = A.mesh.nE * NN;
      double cur[HF][5], nxt[HF][5];
#pragma unroll
      for (int h = 0; h < HF; ++h)
#pragma unroll
        for (int v = 0; v < 5; ++v) cur[h][v] = su[h][v];
#pragma unroll 1
      for (int q = 0; q < FL; ++q) {
        const LineTask<N> t = face_line<N>(lane, q), tn = face_line<N>(lane, q + 1 < FL ? q + 1 : q);
        if (FL > 1)
#pragma unroll
          for (int h = 0; h < HF; ++h) fetch_end<N>(A.U, stride, pl, e, tn, h, nxt[h]);
#pragma unroll
        for (int h = 0; h < HF; ++h) {
          face(t, h, cur[h]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (FL > 1)
#pragma unroll
          for (int h = 0; h < HF; ++h)
#pragma unroll
            for (int v = 0; v < 5; ++v) cur[h][v] = nxt[h][v];
      }
    } else {
#pragma unroll
      for (int q = 0; q < FL; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) face(face_line<N>(lane, q), h, sn[q][h]);
    }
  } else {
    if constexpr (HF == 1) {
      face(LineTask<N>(again(wtid)), 1, su[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    const LineArgs& A = again(args);
    const LineTask<N> t(again(wtid));
    constexpr int NQ = EC && MIXED ? 7 : 6;
    R q[NQ][NP];  // the fields 0..5 (6), velocities in the line frame
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int l = t.node(m);
      q[0][m] = sF[l];
      q[1][m] = sF[(1 + t.d) * EB + l];
      q[2][m] = sF[(1 + t.d1) * EB + l];
      q[3][m] = sF[(1 + t.d2) * EB + l];
      q[4][m] = sF[4 * EB + l];
      q[5][m] = sF[5 * EB + l];
      if constexpr (NQ == 7) q[NQ - 1][m] = sF[6 * EB + l];
    }
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int m = 0; m < NP; ++m) acc[v][m] = R(0);
    if constexpr (!EC) {
      // Kennedy-Gruber pairs of half values: with the sums (means) rho, u, v, w,
      // p, e, f = (m, m u + p, m v, m w, u (rho e + p + p0)), m = rho u; in FP64 p
      // is relative to the line's first node (p0): the multiple of the row sum
      // of Q it leaves out of the momentum vanishes, and so do its rounding errors
      const R ph0 = MIXED ? R(0) : q[4][0], p0 = ph0 + ph0;
      if (!MIXED)
#pragma unroll
        for (int m = 0; m < NP; ++m) q[4][m] -= ph0;
      const auto pair = [&](int i, int m, R (&f)[5]) {
        const R rho = q[0][i] + q[0][m], un = q[1][i] + q[1][m], pm = q[4][i] + q[4][m];
        f[0] = rho * un;
        f[1] = f[0] * un + pm;
        f[2] = f[0] * (q[2][i] + q[2][m]);
        f[3] = f[0] * (q[3][i] + q[3][m]);
        f[4] = un * (rho * (q[5][i] + q[5][m]) + (MIXED ? pm : pm + p0));
      };
#pragma unroll
      for (int dist = N; dist > 0; --dist) {
#pragma unroll
        for (int s = 0; s <= N - dist; ++s) {
          const int i = pair_low(NP - dist, s), m = i + dist;
          R f[5];
          pair(i, m, f);
          const R c = q_im<N, R>(A.basis, i, m);
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            acc[v][i] += c * f[v];
            acc[v][m] -= c * f[v];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (MIXED) {  // strong form at the ends: their own flux
        R f[5];
        pair(0, 0, f);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][0] -= R(0.5) * f[v];
        pair(N, N, f);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][N] += R(0.5) * f[v];
      }
    } else {
      // entropy-conserving pairs.  f of the largest pair is that of the line's
      // extremes: where it is small for rho and beta on every line of the wave,
      // all logarithmic means take their series (the usual case)
      const R two_ref = MIXED ? static_cast<R>(2.0 * sW[NP + 2]) : R(0);
      R lo[2] = {q[0][0], q[4][0]}, hi[2] = {q[0][0], q[4][0]};
#pragma unroll
      for (int m = 1; m < NP; ++m) {
        lo[0] = q[0][m] < lo[0] ? q[0][m] : lo[0];
        hi[0] = q[0][m] > hi[0] ? q[0][m] : hi[0];
        lo[1] = q[4][m] < lo[1] ? q[4][m] : lo[1];
        hi[1] = q[4][m] > hi[1] ? q[4][m] : hi[1];
      }
      // (sqrt of the bounds on f^2: the short series 1e-4, the long one, also that of
      // mixed precision, 1e-2)
      const R dr = hi[0] - lo[0], sr = hi[0] + lo[0], db = hi[1] - lo[1], sb = two_ref + (hi[1] + lo[1]);
      const bool mid = dr >= R(0.01) * sr || db >= R(0.01) * sb;
      const bool large = dr >= R(0.1) * sr || db >= R(0.1) * sb;
      // (momentum relative to the pressure of the line's first node, as above)
      const R pl0 = MIXED ? R(0) : static_cast<R>(q[0][0] * rcp_nr(q[4][0]));
      const R k2 = static_cast<R>((MIXED ? 0.5 : 1.0) / A.ph.gm1);
      const R br = R(0.5) * two_ref, ibr = MIXED ? static_cast<R>(1.0 / sW[NP + 2]) : R(0);
      const auto pair = [&](int i, int m, R (&f)[5]) {
        if constexpr (MIXED) {
          R a[7], b[7];
#pragma unroll
          for (int c = 0; c < 7; ++c) {
            a[c] = q[c][i];
            b[c] = q[c][m];
          }
          ec_pair_ref<true>(a, b, k2, br, ibr, f);
        } else {
          const double sr = q[0][i] + q[0][m], sb = q[4][i] + q[4][m];  // {{rho}}, 2 {{beta}}
          const double x = rcp_nr(sr * sb);
          const double ir = sb * x, ib = sr * x;
          const double fr = (q[0][i] - q[0][m]) * ir, fb = (q[4][i] - q[4][m]) * ib;
          const double ur = fr * fr, ub = fb * fb;
          const double G = 1.0 - ur * (1.0 / 3.0 + ur * (4.0 / 45.0 + ur * (44.0 / 945.0)));
          const double F = 1.0 + ub * (1.0 / 3.0 + ub * (0.2 + ub * (1.0 / 7.0)));
          const double p_hat = sr * ib;
          const double un = q[1][i] + q[1][m], v = q[2][i] + q[2][m], w = q[3][i] + q[3][m];
          f[0] = sr * G * un;
          f[1] = f[0] * un + (p_hat - pl0);
          f[2] = f[0] * v;
          f[3] = f[0] * w;
          f[4] = f[0] * (k2 * ib * F - (q[5][i] + q[5][m]) + (un * un + v * v + w * w)) + p_hat * un;
        }
      };
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(large) != 0, 0)) {
        ec_rows<N, R, false>(A, sF, head, t, static_cast<double>(pl0), acc);
      } else if (!MIXED && __builtin_amdgcn_ballot_w64(mid) != 0) {
        ec_rows<N, R, true>(A, sF, head, t, static_cast<double>(pl0), acc);
      } else {
        settle(q);  // (nothing of the versions is shared, and held, before the branch)
#pragma unroll
        for (int dist = N; dist > 0; --dist) {
#pragma unroll
          for (int s = 0; s <= N - dist; ++s) {
            const int i = pair_low(NP - dist, s), m = i + dist;
            R f[5];
            pair(i, m, f);
            const R c = q_im<N, R>(A.basis, i, m);
#pragma unroll
            for (int v = 0; v < 5; ++v) {
              acc[v][i] += c * f[v];
              acc[v][m] -= c * f[v];
            }
            if (s % 2) __builtin_amdgcn_sched_barrier(0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (MIXED) {
        R f[5];
        pair(0, 0, f);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][0] -= R(0.5) * f[v];
        pair(N, N, f);
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][N] += R(0.5) * f[v];
      }
    }
    settle(acc);
  }
  phase_end();

  // ---- line phase: gradients ------------------------------------------------
  R fn[FACE ? FL : 2][3];  // face lanes: (line, end); line lanes: (end, component)
  R dun[NP], fs[2][5];     // mixed precision: sum D u / 2; surface terms (N = 7)
  R fv[3][NP];             // viscous sums, where they are added apart (SPLIT)
  if constexpr (!FACE) {
    const LineArgs& A = again(args);
    const LineTask<N> t(again(wtid));
    const int nb[2] = {pl.neighbour(t.d, 0), pl.neighbour(t.d, 1)};
    R gh[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int c = 0; c < 3; ++c) gh[h][c] = sF[Fd::end_at(t.d, 8 * h + c, t.ab)];
      if (!MIXED || L::UNIFORM)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const R s = sF[Fd::end_at(t.d, 8 * h + 3 + v, t.ab)];
          if (MIXED)
            fs[h][v] = s;
          else
            acc[v][h ? N : 0] += s;
        }
    }
    if (L::UNIFORM) wave_reuse();  // (the ends' values lie in the gradient fields)
    if (VISC) {
      // the neighbours' normal viscous flux at the ends, in flight over the next phases
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const R* src = static_cast<const R*>(A.ffv) + static_cast<long long>(nb[h] >= 0 ? nb[h] : e) * (6 * 4 * NF) +
                       (2 * t.d + 1 - h) * (4 * NF);
        const unsigned ab = t.ab;
        fn[h][0] = load_once(&(src + t.d * NF)[ab]);
        fn[h][1] = load_once(&(src + t.d1 * NF)[ab]);
        fn[h][2] = load_once(&(src + t.d2 * NF)[ab]);
      }
      // (tangential components at a wall-model wall: the modelled stress)
      if (A.mesh.tauw != nullptr && pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (nb[h] < 0) {
            const double* tw = A.mesh.tauw + wall_face_index(A.mesh, pl.ex, pl.ey, pl.ez, t.d, h != 0) * 3 * NF + t.ab;
            fn[h][1] = static_cast<R>(tw[t.d1 * NF]);
            fn[h][2] = static_cast<R>(tw[t.d2 * NF]);
          }
    }
    if (VISC || MIXED) {
      int ad[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) ad[m] = t.node(m);
#pragma unroll
      for (int c = 0; c < (VISC ? 3 : 1); ++c) {
        const int qc = c == 0 ? t.d : (c == 1 ? t.d1 : t.d2);
        R q[NP], g[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) q[m] = sF[(1 + qc) * EB + ad[m]];
        if (MIXED) {
          line_derivative<N, R, true>(A.basis, q, R(0), R(0), g);
          if (c == 0)
#pragma unroll
            for (int m = 0; m < NP; ++m) dun[m] = g[m];
          g[0] -= R(0.5) * gh[0][c];
          g[N] += R(0.5) * gh[1][c];
        } else {
          line_derivative<N, R, false>(A.basis, q, gh[0][c], gh[1][c], g);
        }
        if (VISC)
#pragma unroll
          for (int m = 0; m < NP; ++m) sF[(GS + 3 * qc + t.d) * EB + ad[m]] = g[m];
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
        fn[q][h] = load_once(&(static_cast<const R*>(A.ffv) + static_cast<long long>(nb[h] >= 0 ? nb[h] : e) * (6 * 4 * NF) +
                               ((2 * t.d + 1 - h) * 4 + 3) * NF)[static_cast<unsigned>(t.ab)]);
      R T[NP], g[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) T[m] = sF[Fd::TS * EB + t.node(m)];
      if constexpr (!Fd::KEEP_T)
#pragma unroll
        for (int h = 0; h < 2; ++h) gt[h] = sF[Fd::GT + h * L::LINES + t.d * NF + t.ab];
      line_derivative<N, R, MIXED>(A.basis, T, gt[0], gt[1], g);
      const double sk = 0.5 * A.ph.kappa * (t.d == 0 ? pl.sx : (t.d == 1 ? pl.sy : pl.sz));
#pragma unroll
      for (int m = 0; m < NP; ++m) g[m] *= static_cast<R>(sk * A.basis.inv_w[m]);
      if (A.ph.suth)
#pragma unroll
        for (int m = 0; m < NP; ++m) g[m] *= sF[Fd::MU + t.node(m)];
      const R qw = pick3(A.mesh.bc[0], A.mesh.bc[1], A.mesh.bc[2], t.d) == DG_BC_WALL_MODEL ? R(-1) : R(1);
      line_derivative<N, R, false>(A.basis, g, (nb[0] < 0 ? qw : R(0)) * g[0], (nb[1] < 0 ? qw : R(0)) * g[N], eh[q]);
    }
    settle(eh);
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
          const R c0 = static_cast<R>(pl.sx * sW[i]), c1 = static_cast<R>(pl.sy * sW[j]), c2 = static_cast<R>(pl.sz * sW[k]);
          R mu = static_cast<R>(A.ph.mu);  // half fluxes: the gradients are those of half velocities
          if (A.ph.suth) mu *= sF[Fd::MU + l];
          R gr[9];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            gr[3 * c] = c0 * sF[(GS + 3 * c) * EB + l];
            gr[3 * c + 1] = c1 * sF[(GS + 1 + 3 * c) * EB + l];
            gr[3 * c + 2] = c2 * sF[(GS + 2 + 3 * c) * EB + l];
          }
          const R dd = R(2.0 / 3.0) * (gr[0] + gr[4] + gr[8]);
          const R t00 = mu * (gr[0] + gr[0] - dd), t11 = mu * (gr[4] + gr[4] - dd), t22 = mu * (gr[8] + gr[8] - dd);
          const R t01 = mu * (gr[1] + gr[3]), t02 = mu * (gr[2] + gr[6]), t12 = mu * (gr[5] + gr[7]);
          const R uu = R(2) * sF[EB + l], vv = R(2) * sF[2 * EB + l], ww = R(2) * sF[3 * EB + l];
          sF[GS * EB + l] = t00;
          sF[(GS + 1) * EB + l] = t11;
          sF[(GS + 2) * EB + l] = t22;
          sF[(GS + 3) * EB + l] = t01;
          sF[(GS + 4) * EB + l] = t02;
          sF[(GS + 5) * EB + l] = t12;
          sF[(GS + 6) * EB + l] = uu * t00 + vv * t01 + ww * t02;
          sF[(GS + 7) * EB + l] = uu * t01 + vv * t11 + ww * t12;
          sF[(GS + 8) * EB + l] = uu * t02 + vv * t12 + ww * t22;
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
      // tau_qd: the diagonal at GS + d, (0,1), (0,2), (1,2) at GS + 2 + q + d
      const int qc = c == 1 ? t.d1 : t.d2;
      const int slot = c == 0 ? GS + t.d : GS + 2 + qc + t.d;
      R f[NP], g[NP], gw[2];
#pragma unroll
      for (int m = 0; m < NP; ++m) f[m] = sF[slot * EB + ad[m]];
      // ghosts: half the neighbour's flux; at a wall 2 f* - f: the own stresses at
      // an isothermal no-slip wall; the own normal stress and the modelled shear
      // stress at a wall-model wall
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool wall = nb[h] < 0;
        const R of_n = !wall ? R(0.5) : (wm && c > 0 ? (h ? R(-1) : R(1)) : R(0));
        const R of_o = !wall ? R(0) : (wm && c > 0 ? R(-1) : R(1));
        gw[h] = of_n * fn[h][c] + of_o * f[h ? N : 0];
      }
      line_derivative<N, R, false>(A.basis, f, gw[0], gw[1], g);
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        if (Fd::SPLIT)
          fv[c][m] = g[m];
        else
          acc[1 + c][m] -= g[m];
      }
    }
    if (Fd::SPLIT)
      settle(fv);
    else
      settle(acc);
  } else if constexpr (VISC) {
    // the stresses' work, u . tau_d (a wall's own does no work: ghost -f)
    const LineArgs& A = again(args);
    const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
    for (int q = 0; q < FL; ++q) {
      const LineTask<N> t = face_line<N>(lane, q);
      R f[NP], g[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) f[m] = sF[(GS + 6 + t.d) * EB + t.node(m)];
      const R g0 = pl.neighbour(t.d, 0) < 0 ? -f[0] : R(0.5) * fn[q][0];
      const R g1 = pl.neighbour(t.d, 1) < 0 ? -f[N] : R(0.5) * fn[q][1];
      line_derivative<N, R, false>(A.basis, f, g0, g1, g);
#pragma unroll
      for (int m = 0; m < NP; ++m) eh[q][m] += g[m];
    }
    settle(eh);
  }

  __builtin_amdgcn_sched_barrier(0);
  // ---- sums of the three directions, scaling, output -----------------------
  const auto viscous_sums = [&](const LineTask<N>& t) {
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      R* o = sF + (Fd::VS + 3 * t.d) * EB + t.node(m);
      o[t.d * EB] = fv[0][m];
      o[t.d1 * EB] = fv[1][m];
      o[t.d2 * EB] = fv[2][m];
    }
  };
  phase_end();
  if constexpr (!FACE) {
    const LineTask<N> t(again(wtid));
    R* o = sF + (MIXED ? 4 : 5) * t.d * EB;
    const double p_ref = MIXED ? sW[NP] : 0.0, e_ref = MIXED ? sW[NP + 1] : 0.0;
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int l = t.node(m);
      if (MIXED)
        reinterpret_cast<double*>(sF + (12 + 2 * t.d) * EB)[l] =
            static_cast<double>(acc[4][m]) + e_ref * static_cast<double>(acc[0][m]) + p_ref * static_cast<double>(dun[m]);
      else
        o[4 * EB + l] = acc[4][m];
      o[l] = acc[0][m];
      o[(1 + t.d) * EB + l] = acc[1][m];
      o[(1 + t.d1) * EB + l] = acc[2][m];
      o[(1 + t.d2) * EB + l] = acc[3][m];
    }
    if (MIXED && L::UNIFORM)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const int k = v == 1 ? 1 + t.d : (v == 2 ? 1 + t.d1 : (v == 3 ? 1 + t.d2 : v));
          sF[Fd::surface_at(t.d, h, k, t.ab)] = fs[h][v];
        }
    if (Fd::SPLIT && !Fd::TWICE && VISC) viscous_sums(t);
  } else if constexpr (VISC) {
    const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
    for (int q = 0; q < FL; ++q) {
      const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
      for (int m = 0; m < NP; ++m) sF[((MIXED ? 18 : 15) + t.d) * EB + t.node(m)] = eh[q][m];
    }
  }
  phase_end();
  double ut[ROUNDS][5];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const unsigned n = node_of<N>(tl, r);
    const int i = n % NP, j = (n / NP) % NP, k = n / NF;
    const int l = L::at(i, j, k);
    const double c[3] = {-2.0 * (pl.sx * sW[i]), -2.0 * (pl.sy * sW[j]), -2.0 * (pl.sz * sW[k])};
#pragma unroll
    for (int v = 0; v < 5; ++v) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double f;
        if (!MIXED)
          f = sF[(5 * d + v) * EB + l];
        else if (v < 4)
          f = sF[(4 * d + v) * EB + l];
        else
          f = reinterpret_cast<const double*>(sF + (12 + 2 * d) * EB)[l];
        if (VISC && v == 4) f -= static_cast<double>(sF[((MIXED ? 18 : 15) + d) * EB + l]);
        ut[r][v] = d == 0 ? c[0] * f : ut[r][v] + c[d] * f;
      }
    }
    if constexpr (MIXED) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int x = d == 0 ? i : (d == 1 ? j : k);
        if (x == 0 || x == N) {
          const int ab = d == 0 ? j + NP * k : (d == 1 ? i + NP * k : i + NP * j);
          const R* o = sF + Fd::surface_at(d, x == N ? 1 : 0, 0, ab);
          // (in the faces' place components are in the line frame: 0, along, across, 4)
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            const int w = L::UNIFORM || v % 4 == 0 ? v : 1 + (v - 1 - d + 3) % 3;
            ut[r][v] += c[d] * static_cast<double>(o[w * L::LINES]);
          }
        }
      }
    }
  }
  if constexpr (Fd::SPLIT && VISC) {
    if constexpr (Fd::TWICE) {
      settle(ut);
      phase_end();
      if constexpr (!FACE) viscous_sums(LineTask<N>(again(wtid)));
      phase_end();
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const unsigned n = node_of<N>(tl, r);
      const int i = n % NP, j = (n / NP) % NP, k = n / NF;
      const R* o = sF + Fd::VS * EB + L::at(i, j, k);
      const double c[3] = {2.0 * (pl.sx * sW[i]), 2.0 * (pl.sy * sW[j]), 2.0 * (pl.sz * sW[k])};
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = 0; v < 3; ++v) ut[r][1 + v] += c[d] * static_cast<double>(o[(3 * d + v) * EB]);
    }
  }
  double g1[ROUNDS][5], u1[ROUNDS][5];  // Ut or the new G, and the new U
  {
    const LineArgs& A = again(args);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        if (RK) {
          g1[r][v] = A.st.read_G ? A.st.A * gA[r][v] + A.st.dt * ut[r][v] : A.st.dt * ut[r][v];
          u1[r][v] = u[r][v] + A.st.B * g1[r][v];
        } else {
          g1[r][v] = ut[r][v];
        }
      }
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
}

template <int N, typename R, bool RK, bool VISC, bool EC>
__global__ __launch_bounds__(Line<N>::BS) __attribute__((amdgpu_waves_per_eu(line_waves<N, R, EC>()))) void k_rhs_line(LineArgs) {
  using L = Line<N>;
  extern __shared__ double lds[];
  const LineArgsPtr args = (LineArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x, blk = static_cast<int>(blockIdx.x);
  const int e = xcd_remap(blk, gridDim.x);
  // line lane number of this lane; face lanes are those of the last FW waves.  At
  // N = 7 which of the four waves that is changes from workgroup to workgroup, so
  // that not all face waves share a SIMD.
  const int turn = L::UNIFORM ? ((blk >> 3) + (blk >> 8)) & 3 : 0;
  const int wtid = L::UNIFORM ? (tid + 64 * turn) & 255 : tid;
  if (__builtin_amdgcn_readfirstlane(wtid) >= 64 * L::LW)
    rhs_line_phases<N, R, RK, VISC, EC, true>(args, lds, e, tid, wtid);
  else
    rhs_line_phases<N, R, RK, VISC, EC, false>(args, lds, e, tid, wtid);
}

template <int N, typename R, bool EC, bool RK>
hipError_t line_n(const LineArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.mesh.nE)), block(Line<N>::BS);
  const size_t lds = Fields<N, R, EC>::bytes(a.ph);
  if (a.ph.viscous)
    hipLaunchKernelGGL((k_rhs_line<N, R, RK, true, EC>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((k_rhs_line<N, R, RK, false, EC>), grid, block, lds, s, a);
  return hipGetLastError();
}

template <typename R, bool EC>
hipError_t line_dispatch(int N, bool rk, const LineArgs& a, hipStream_t s) {
  switch (N) {
    case 3: return rk ? line_n<3, R, EC, true>(a, s) : line_n<3, R, EC, false>(a, s);
    case 5: return rk ? line_n<5, R, EC, true>(a, s) : line_n<5, R, EC, false>(a, s);
    case 7: return rk ? line_n<7, R, EC, true>(a, s) : line_n<7, R, EC, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace dg
