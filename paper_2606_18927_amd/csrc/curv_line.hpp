// Right-hand side (and fused RK stage) on curvilinear elements with line lanes,
// for gfx950: the phases of line_device.hpp, with metric terms.
//
//   nodes  primitives of U into LDS;
//   lines  line lanes: contravariant two-point fluxes of the line's pairs, with the
//          averaged metric vector (J a^d(i) + J a^d(m)) / 2 of the line's direction d, once
//          per pair; face lanes: surface fluxes with the face normal J a^d (that of the
//          element below the face, shared by both sides), ghost values;
//   lines  derivatives of u, v, w (line lanes) and T (face lanes) along the line;
//   nodes  physical gradients (1/J) sum_r J a^r D_r q, stress and heat flux, the contravariant
//          viscous fluxes of the three directions, in place;
//   lines  their derivatives (momentum: line lanes, energy: face lanes);
//   nodes  the three directions' sums, Ut = -(1/J) (...), output or RK update.
//
// What bounds it (N = 7, 32^3 elements, RK instance, per launch; with one lane per node
// in brackets): Kennedy-Gruber pair FP64 1245 us (1590), 5.39 GB of HBM traffic (5.84),
// vector instructions issue 40 % of the time; mixed 943 us (1290), 5.27 GB, 69 %;
// entropy-conserving pair FP64 1419 us (2860), mixed 1190 us (1750), 87 %.  A triad moves
// 5.3 GB in 0.83 ms: the metric terms, ten values per node against five of the state, are
// most of the traffic.  FP64 holds two workgroups per CU (81 KB LDS), mixed three.
//
// Summation by parts takes the surface terms as in line_device.hpp.  Mixed precision
// (FP32 LDS fields, gradients, metric terms of the sweeps, fluxes and line sums; p, e and T,
// or beta and pi, relative to the element's first node) keeps the strong form at the faces:
// surface flux minus own flux in FP64, added to the sums in FP64 at the end, as the
// viscous sums of the momentum and the energy are; the reference pressure's share of the momentum sums is the discrete divergence of the
// metric terms (zero) and is dropped, the energy's e_ref sum D (rho U~)# + p_ref sum D U~#
// is added back in FP64.
#pragma once

#include "curv_flux.hpp"
#include "line_device.hpp"

namespace dg {
namespace {

// LDS fields (of EB values of type R), as Fields with all twelve gradient components
// GS + 3 q + r (q = u, v, w, T; r the line direction), then the contravariant half viscous
// fluxes GS + 3 c + r in their place.
template <int N, typename R, bool EC>
struct CurvFields {
  using L = Line<N>;
  static constexpr bool MIXED = sizeof(R) == 4;
  static constexpr int NQ = EC && MIXED ? 7 : 6;  // rho, u, v, w, p, e | beta, |u|^2 / 4 (, pi / 2)
  static constexpr int TS = NQ, GS = TS + 1;
  static constexpr int COUNT = MIXED ? 21 : GS + 12;
  static constexpr int ENDS = COUNT * L::EB;
  static constexpr int GT = ENDS + (L::UNIFORM ? 0 : 16 * L::LINES);
  static constexpr int OWN = (L::UNIFORM ? GS + 6 : GS) * L::EB;  // 5 FP64 values per boundary node
  static constexpr int NB = n_face_nodes<N>();
  static_assert(!MIXED || OWN + 10 * NB <= (GS + 12) * L::EB, "boundary states fit");
  static_assert(!MIXED || 20 * L::LINES + 9 * L::EB <= COUNT * L::EB + (L::UNIFORM ? 0 : 16 * L::LINES),
                "the faces' FP64 terms and the viscous sums fit");
  static constexpr int HEAD = 16;  // FP64: 1 / w_i, then p_ref, e_ref, beta_ref, T_ref
  // faces of a line that its face lane takes (line_faces; mixed precision holds their FP64 terms)
  static constexpr int HF = line_faces<N, EC || (MIXED && N == 7)>();
  // Ghost temperatures in the face lane's registers (as Fields), except where registers and
  // not LDS bound the workgroups of a CU (N = 5 entropy-conserving in FP64: 3 % slower so).
  static constexpr bool KEEP_T = !L::UNIFORM && HF == 2 && (MIXED || !EC);
  static constexpr size_t BYTES =
      HEAD * sizeof(double) + sizeof(R) * static_cast<size_t>(GT + (KEEP_T ? 0 : 2 * L::LINES));
  // Nodes of a line held in registers, and the waves per SIMD that the registers are bounded
  // for: what LDS lets a CU hold, unless the bound spills more than a few values.  N = 5 in
  // FP64 fits a third workgroup with half lines (16^3 elements: 590 -> 535 us a step), mixed
  // entropy-conserving a fourth (density noise of 0.1 / 40 %: 616 -> 573, 1071 -> 1011 us).
  // Entropy-conserving in FP64, N = 3 spills 38 for a third (24^3: 804 -> 755, 1347 -> 1495).
  static constexpr int BLOCK = N == 7 ? 4 : (N == 5 && !MIXED && !EC ? 3 : L::NP);
  static constexpr int WAVES = MIXED ? (N == 7 || (N == 3 && EC) ? 3 : 4) : (N == 7 || EC ? 2 : (N == 5 ? 3 : 4));
  __device__ static int end_at(int d, int k, int ab) {
    return L::UNIFORM ? (GS + 3 * (k >> 3) + d) * L::EB + (k & 7) * L::NF + ab : ENDS + k * L::LINES + d * L::NF + ab;
  }
};

template <typename R>
struct FaceReads {  // (fetch_face)
  static constexpr int COUNT = sizeof(R) == 8 ? 11 : 8;
};

// Metric component c at node idx in the sweep precision: FP64 or its FP32 copy, stored
// after the ten FP64 fields.
template <typename R>
__device__ inline const R* geo_field(const DevMesh& m, long long stride, int c) {
  if constexpr (sizeof(R) == 4)
    return reinterpret_cast<const float*>(m.geo + 10 * stride) + c * stride;
  else
    return m.geo + c * stride;
}

// The two-point flux of a pair from halves of (rho, u, v, w, p, e) and of the metric
// vectors: f = (m, m u_c + p M_c, m e + p U~), U~ = u . M, m = rho U~; f[5] = U~.
template <typename R>
__device__ __forceinline__ void kg_contra(const R* a, const R (&Ma)[3], const R* b, const R (&Mb)[3], R (&f)[6]) {
  const R M0 = Ma[0] + Mb[0], M1 = Ma[1] + Mb[1], M2 = Ma[2] + Mb[2];
  const R rho = a[0] + b[0], u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3], p = a[4] + b[4], e = a[5] + b[5];
  f[5] = u * M0 + v * M1 + w * M2;
  f[0] = rho * f[5];
  f[1] = f[0] * u + p * M0;
  f[2] = f[0] * v + p * M1;
  f[3] = f[0] * w + p * M2;
  f[4] = f[0] * e + p * f[5];
}

// Chandrashekar's pair in FP64, x = (rho, u, v, w) / 2, beta, |u|^2 / 4; MEANS 0: short
// series (f^2 below 1e-4), 1: long series (1e-2), 2: chosen.
template <int MEANS>
__device__ __forceinline__ void ec_contra(const double* a, const double (&Ma)[3], const double* b, const double (&Mb)[3],
                                          double k2, double (&f)[6]) {
  const double M0 = Ma[0] + Mb[0], M1 = Ma[1] + Mb[1], M2 = Ma[2] + Mb[2];
  const double sr = a[0] + b[0], sb = a[4] + b[4];
  const double x = rcp_nr(sr * sb), ir = sb * x, ib = sr * x;
  const double fr = (a[0] - b[0]) * ir, fb = (a[4] - b[4]) * ib;
  const double ur = fr * fr, ub = fb * fb;
  double G, F;
  if constexpr (MEANS == 1) {
    double unused;
    ln_series(ur, unused, G);
    ln_series(ub, F, unused);
  } else {
    G = 1.0 - ur * (1.0 / 3.0 + ur * (4.0 / 45.0 + ur * (44.0 / 945.0)));
    F = 1.0 + ub * (1.0 / 3.0 + ub * (0.2 + ub * (1.0 / 7.0)));
    if constexpr (MEANS == 2) {
      if (ur >= 1e-4) G = fr / atanh(fr);
      if (ub >= 1e-4) F = atanh(fb) / fb;
    }
  }
  const double p = sr * ib, u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3];
  f[5] = u * M0 + v * M1 + w * M2;
  f[0] = sr * G * f[5];
  f[1] = f[0] * u + p * M0;
  f[2] = f[0] * v + p * M1;
  f[3] = f[0] * w + p * M2;
  f[4] = f[0] * (k2 * ib * F - (a[5] + b[5]) + (u * u + v * v + w * w)) + p * f[5];
}

// The same in FP32 relative to the element's reference state (ec_pair_ref's means);
// MEANS 0: series (f^2 below 1e-2), 2: chosen.
template <int MEANS>
__device__ __forceinline__ void ec_contra_ref(const float* a, const float (&Ma)[3], const float* b, const float (&Mb)[3],
                                              float kap, float beta_ref, float ibr, float (&f)[6]) {
  const float M0 = Ma[0] + Mb[0], M1 = Ma[1] + Mb[1], M2 = Ma[2] + Mb[2];
  const float sr = a[0] + b[0], sdb = a[4] + b[4], sb = 2.0f * beta_ref + sdb;
  const float x = __builtin_amdgcn_rcpf(sr * sb), ir = sb * x, ib = sr * x;
  const float fr = (a[0] - b[0]) * ir, fb = (a[4] - b[4]) * ib;
  const float ur = fr * fr, ub = fb * fb;
  float G = 1.0f - ur * (1.0f / 3.0f + ur * (4.0f / 45.0f + ur * (44.0f / 945.0f)));
  float Fs = ub * (1.0f / 3.0f + ub * (0.2f + ub * (1.0f / 7.0f)));
  if constexpr (MEANS == 2) {
    if (ur >= 1e-2f) G = fr / atanhf(fr);
    if (ub >= 1e-2f) Fs = atanhf(fb) / fb - 1.0f;
  }
  const float u = a[1] + b[1], v = a[2] + b[2], w = a[3] + b[3];
  f[5] = u * M0 + v * M1 + w * M2;
  f[0] = sr * G * f[5];
  const float dp = (a[6] + b[6]) * ib;
  f[1] = f[0] * u + dp * M0;
  f[2] = f[0] * v + dp * M1;
  f[3] = f[0] * w + dp * M2;
  f[4] = f[0] * (kap * ((2.0f * Fs - sdb * ibr) * ib) - (a[5] + b[5]) + (u * u + v * v + w * w)) + dp * f[5];
}

template <int N, typename R, bool EC, int MEANS>
__device__ __forceinline__ void curv_pair(const DevPhys& ph, const double* head, const R* a, const R (&Ma)[3], const R* b,
                                          const R (&Mb)[3], R (&f)[6]) {
  if constexpr (!EC)
    kg_contra<R>(a, Ma, b, Mb, f);
  else if constexpr (sizeof(R) == 4)
    ec_contra_ref<MEANS>(a, Ma, b, Mb, static_cast<float>(0.5 / ph.gm1), static_cast<float>(head[N + 3]),
                         static_cast<float>(1.0 / head[N + 3]), f);
  else
    ec_contra<MEANS>(a, Ma, b, Mb, 1.0 / ph.gm1, f);
}

// acc[v][i] = sum_{m != i} Q_im f_v(i, m), unrolled; M: halves of the line's metric vectors.
// (FP64 lines of eight nodes, their metrics and sums exceed the registers: blocks of
// four, the second block's nodes one by one against the first.)
template <int N, typename R, bool EC, int NV>
__device__ __forceinline__ void curv_pairs(const LineArgs& A, const R* sF, const double* head, const LineTask<N>& t,
                                           const R (&M)[N + 1][3], R (&acc)[NV][N + 1]) {
  using Fd = CurvFields<N, R, EC>;
  constexpr int NP = N + 1, H = Fd::BLOCK, NQ = Fd::NQ, EB = Line<N>::EB;
  R x[H][NQ];
  const auto load = [&](int m, R* q) {
    const int l = t.node(m);
#pragma unroll
    for (int c = 0; c < NQ; ++c) q[c] = sF[c * EB + l];
  };
  const auto pair = [&](const R* a, int i, const R* b, int m) {
    R f[6];
    curv_pair<N, R, EC, 0>(A.ph, head, a, M[i], b, M[m], f);
    const R c = q_im<N, R>(A.basis, i, m);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      acc[v][i] += c * f[v];
      acc[v][m] -= c * f[v];
    }
  };
  if constexpr (!Fd::MIXED) {
#pragma unroll
    for (int b0 = 0; b0 < NP; b0 += H) {
#pragma unroll
      for (int i = 0; i < H; ++i) load(b0 + i, x[i]);
      if (EC) settle(x);  // (nothing of this and the rolled version is shared before the branch)
#pragma unroll
      for (int i = 0; i < H; ++i)
#pragma unroll
        for (int m = i + 1; m < H; ++m) {
          pair(x[i], b0 + i, x[m], b0 + m);
          if (EC || m % 2) __builtin_amdgcn_sched_barrier(0);
        }
      if (b0 == 0)
#pragma unroll
        for (int m = H; m < NP; ++m) {
          R z[NQ];
          load(m, z);
#pragma unroll
          for (int i = 0; i < H; ++i) {
            pair(x[i], i, z, m);
            if (EC || i % 2) __builtin_amdgcn_sched_barrier(0);
          }
        }
    }
  } else {  // from the farthest pairs to the nearest (pair_low), the second block mirrored
    const auto block = [&](int b0) {
#pragma unroll
      for (int dist = H - 1; dist > 0; --dist)
#pragma unroll
        for (int s = 0; s < H - dist; ++s) {
          const int k = pair_low(H - dist, s), i = b0 ? H - 1 - dist - k : k;
          pair(x[i], b0 + i, x[i + dist], b0 + i + dist);
          if (EC || s % 2) __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int i = 0; i < H; ++i) load(i, x[i]);
    if (EC) settle(x);
    if (EC) block(0);  // (last, its pairs spill twice as many registers)
#pragma unroll
    for (int m = N; m >= H; --m) {
      R z[NQ];
      load(m, z);
#pragma unroll
      for (int i = 0; i < H; ++i) {
        pair(x[i], i, z, m);
        if (EC || i % 2) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (!EC) block(0);
    if constexpr (H < NP) {
#pragma unroll
      for (int i = 0; i < H; ++i) load(NP - H + i, x[i]);
      if (EC) settle(x);
      block(NP - H);
    }
  }
}

// The same for states with larger jumps, not unrolled.
template <int N, typename R, int MEANS, int NV>
__device__ inline void curv_rows(const LineArgs& A, const R* sF, const double* head, const LineTask<N>& t,
                                 const R* geo0, long long stride, R (&acc)[NV][N + 1]) {
  using Fd = CurvFields<N, R, true>;
  constexpr int NP = N + 1, NQ = Fd::NQ, EB = Line<N>::EB;
  const auto load = [&](int m, R* q, R (&M)[3]) {
    const int l = t.node(m);
#pragma unroll
    for (int c = 0; c < NQ; ++c) q[c] = sF[c * EB + l];
#pragma unroll
    for (int c = 0; c < 3; ++c) M[c] = R(0.5) * (geo0 + c * stride)[t.end_node(m)];
  };
#pragma unroll 1
  for (int i = 0; i < N; ++i) {
    R a[NQ], Ma[3], s[NV];
    load(i, a, Ma);
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = R(0);
#pragma unroll 1
    for (int m = N; m > i; --m) {
      R b[NQ], Mb[3], f[6];
      load(m, b, Mb);
      curv_pair<N, R, true, MEANS>(A.ph, head, a, Ma, b, Mb, f);
      const R c = q_im<N, R>(A.basis, i, m);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        f[v] *= c;
        s[v] += f[v];
      }
#pragma unroll
      for (int r = 1; r < NP; ++r) {
        const R sel = r == m ? R(-1) : R(0);
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v][r] += sel * f[v];
      }
    }
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const R sel = r == i ? R(1) : R(0);
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v][r] += sel * s[v];
    }
  }
}

// What a face lane reads of one face: the neighbour's state, the face normal and (FP64, on a
// lower face; on an upper one it is the face normal) the own metric vector there.
template <int N, typename R>
__device__ __forceinline__ void fetch_face(const LineArgs& A, long long stride, const Place& pl, int e, const LineTask<N>& t,
                                           int h, double (&s)[FaceReads<R>::COUNT]) {
  const int nb = pl.neighbour(t.d, h);
  const unsigned on = t.end_node(h ? N : 0), nn = t.end_node(h ? 0 : N);
  const double* p = A.U + static_cast<long long>(nb >= 0 ? nb : e) * Line<N>::NN;
#pragma unroll
  for (int v = 0; v < 5; ++v) s[v] = (p + v * stride)[nn];
  // the normal of the element below the face (a wall: the own), so that the two sides'
  // fluxes are exact negatives
  const bool own = h != 0 || nb < 0;
  const long long ge = own ? e : nb;
  const unsigned gn = own ? on : nn;
  if constexpr (sizeof(R) == 4) {
    // the sweeps read the FP32 copy: the boundary nodes' copy is the smaller fetch
    constexpr int NB = n_face_nodes<N>();
    const unsigned i = gn % (N + 1), j = (gn / (N + 1)) % (N + 1), k = gn / Line<N>::NF;
    const double* g = A.mesh.geoF + ge * NB + face_node_index<N>(i, j, k);
#pragma unroll
    for (int c = 0; c < 3; ++c) s[5 + c] = g[(3 * t.d + c) * (A.mesh.nE * NB)];
  } else {
    const double* g = A.mesh.geo + ge * Line<N>::NN;
#pragma unroll
    for (int c = 0; c < 3; ++c) s[5 + c] = (g + (3 * t.d + c) * stride)[gn];
    if (h == 0) {
      const double* go = A.mesh.geo + static_cast<long long>(e) * Line<N>::NN;
#pragma unroll
      for (int c = 0; c < 3; ++c) s[8 + c] = (go + (3 * t.d + c) * stride)[on];
    }
  }
}

// One face node: the ghost velocities (halves) and temperature, and -+ half the surface
// flux; mixed precision: the jumps to them, and -+ half (surface flux - own flux).
// The weak form drops the own flux with the own metric vector M, where the strong form
// has it with the face normal s on both sides.  The two differ by the rounding of the two
// elements' metric terms, but the flux holds the pressure: f(M - s) is added (without it the
// momentum's rounding error at Ma = 0.1 is 5, 17 and 21 times larger at N = 3, 5, 7).
template <int N, typename R, bool EC>
__device__ __forceinline__ void curv_face(const LineArgs& A, const R* sF, const LineTask<N>& t, int h, bool wall,
                                          const double (&sn)[FaceReads<R>::COUNT], R (&gv)[3], R& gT, double (&fs)[5]) {
  using L = Line<N>;
  using Fd = CurvFields<N, R, EC>;
  constexpr int EB = L::EB;
  const double s[3] = {sn[5], sn[6], sn[7]};
  const double irn = rcp_nr(sn[0]);
  const double vn[3] = {sn[1] * irn, sn[2] * irn, sn[3] * irn};
  const double q2n = vn[0] * vn[0] + vn[1] * vn[1] + vn[2] * vn[2];
  const double pn = A.ph.gm1 * (sn[4] - 0.5 * sn[0] * q2n);
  const double Tn = pn * A.ph.inv_R * irn;
  double so[5], vo[3], po, To, q2o;  // own
  if constexpr (Fd::MIXED) {
    const unsigned a = static_cast<unsigned>(t.ab) % L::NP, b = static_cast<unsigned>(t.ab) / L::NP;
    const int n = h ? N : 0;
    const double* own = reinterpret_cast<const double*>(sF + Fd::OWN) +
                        face_node_index<N>(t.d == 0 ? n : a, t.d == 0 ? a : (t.d == 1 ? n : b), t.d == 2 ? n : b);
#pragma unroll
    for (int v = 0; v < 5; ++v) so[v] = own[v * Fd::NB];
    const double iro = rcp_nr(so[0]);
#pragma unroll
    for (int c = 0; c < 3; ++c) vo[c] = so[1 + c] * iro;
    q2o = vo[0] * vo[0] + vo[1] * vo[1] + vo[2] * vo[2];
    po = A.ph.gm1 * (so[4] - 0.5 * so[0] * q2o);
    To = po * A.ph.inv_R * iro;
#pragma unroll
    for (int c = 0; c < 3; ++c) gv[c] = static_cast<R>(wall ? -vo[c] : 0.5 * (vn[c] - vo[c]));
    gT = static_cast<R>(wall ? 2.0 * (A.mesh.T_wall - To) : Tn - To);
  } else {
    const int l = t.node(h ? N : 0);
    so[0] = 2.0 * sF[l];
#pragma unroll
    for (int c = 0; c < 3; ++c) vo[c] = 2.0 * sF[(1 + c) * EB + l];
    q2o = vo[0] * vo[0] + vo[1] * vo[1] + vo[2] * vo[2];
    if (EC) {
      const double be = sF[4 * EB + l];
      po = quot(0.5 * so[0], be, rcp_nr(be));
      so[4] = po / A.ph.gm1 + 0.5 * so[0] * q2o;
    } else {
      po = 2.0 * sF[4 * EB + l];
      so[4] = so[0] * (2.0 * sF[5 * EB + l]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) so[1 + c] = so[0] * vo[c];
    To = sF[Fd::TS * EB + l];
#pragma unroll
    for (int c = 0; c < 3; ++c) gv[c] = wall ? -0.5 * vo[c] : 0.5 * vn[c];
    gT = wall ? 2.0 * A.mesh.T_wall - To : Tn;
  }
  double F[5];
  const double smag2 = s[0] * s[0] + s[1] * s[1] + s[2] * s[2];
  if constexpr (EC) {
    const double A6[6] = {so[0], vo[0], vo[1], vo[2], quot(0.5 * so[0], po, rcp_nr(po)), q2o};
    const double B6[6] = {sn[0], vn[0], vn[1], vn[2], quot(0.5 * sn[0], pn, rcp_nr(pn)), q2n};
    ec_flux_contra(A6, B6, s[0], s[1], s[2], A.ph.gm1, F);
    if (!A.ph.central) {
      const double smag = sqrt_nr(smag2), ism = rcp_nr(smag);
      const double n[3] = {s[0] * ism, s[1] * ism, s[2] * ism};
      // L = own on an upper face, the neighbour on a lower face
      const double Po[5] = {so[0], vo[0], vo[1], vo[2], po}, Pn[5] = {sn[0], vn[0], vn[1], vn[2], pn};
      double X[5], Y[5], D[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        X[v] = h ? Po[v] : Pn[v];
        Y[v] = h ? Pn[v] : Po[v];
      }
      roe_dissipation_normal(X, h ? so[4] : sn[4], Y, h ? sn[4] : so[4], n, A.ph.gamma, D);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] -= 0.5 * smag * D[v];
    }
  } else {
    const double rho = 0.5 * (so[0] + sn[0]), u = 0.5 * (vo[0] + vn[0]), v = 0.5 * (vo[1] + vn[1]), w = 0.5 * (vo[2] + vn[2]);
    const double p = 0.5 * (po + pn);
    const double iro = rcp_nr(so[0]);
    const double e = 0.5 * (so[4] * iro + sn[4] * irn);
    const double U = u * s[0] + v * s[1] + w * s[2], m = rho * U;
    F[0] = m;
    F[1] = m * u + p * s[0];
    F[2] = m * v + p * s[1];
    F[3] = m * w + p * s[2];
    F[4] = m * e + p * U;
    if (!A.ph.central) {
      const double smag = sqrt_nr(smag2), go = A.ph.gamma * po, gn = A.ph.gamma * pn;
      const double lo = fabs(vo[0] * s[0] + vo[1] * s[1] + vo[2] * s[2]) + sqrt_edge(quot(go, so[0], iro)) * smag;
      const double ln = fabs(vn[0] * s[0] + vn[1] * s[1] + vn[2] * s[2]) + sqrt_edge(quot(gn, sn[0], irn)) * smag;
      const double hl = (h ? 0.5 : -0.5) * (lo >= ln ? lo : ln);
#pragma unroll
      for (int c = 0; c < 5; ++c) F[c] -= hl * (sn[c] - so[c]);
    }
  }
  const double sg = h ? 0.5 : -0.5;
  const double Uo = vo[0] * s[0] + vo[1] * s[1] + vo[2] * s[2];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double ps = v >= 1 && v <= 3 ? po * s[v - 1] : (v == 4 ? po * Uo : 0.0);
    const double wf = v >= 1 && v <= 3 ? ps : 0.0;  // impermeable wall: the interior pressure only
    double own = 0.0;
    if constexpr (Fd::MIXED) {
      own = so[v] * Uo + ps;
    } else if (h == 0) {
      const double m[3] = {s[0] - sn[8], s[1] - sn[9], s[2] - sn[10]};
      const double Um = vo[0] * m[0] + vo[1] * m[1] + vo[2] * m[2];
      own = so[v] * Um + (v >= 1 && v <= 3 ? po * m[v - 1] : (v == 4 ? po * Um : 0.0));
    }
    fs[v] = sg * ((wall ? wf : F[v]) - own);
  }
}

template <int N, typename R, bool RK, bool VISC, bool EC, bool FACE>
__device__ __forceinline__ void curv_phases(const LineArgsPtr args, double* const head, const int e, const int tid,
                                            const int wtid) {
  using L = Line<N>;
  using Fd = CurvFields<N, R, EC>;
  constexpr int NP = L::NP, NF = L::NF, NN = L::NN, EB = L::EB, BS = L::BS, ROUNDS = L::ROUNDS, FL = L::FL, LINES = L::LINES;
  constexpr int GS = Fd::GS, NQ = Fd::NQ;
  constexpr bool MIXED = Fd::MIXED;
  constexpr int NV = MIXED ? 6 : 5;
  double* const sW = head;
  R* const sF = reinterpret_cast<R*>(head + Fd::HEAD);
  const Place pl(again(args).mesh, e, false);
  R eh[FL][NP];             // face lanes: the diffusive part of the lines' energy sums
  constexpr int HF = Fd::HF, FF = FACE ? FL : 1, H0 = FACE ? 0 : HF, H1 = FACE ? HF : 2;  // own faces
  double fe[FF][2][5];      // mixed precision: the faces' parts of the sums
  R acc[NV][NP];            // line lanes: sums of the line's nodes; mixed: [5] sum D U~
  R gt[2];                  // ghost temperatures
  {
    const LineArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
    double u[ROUNDS][5], sn[EC ? 1 : FL][2][FaceReads<R>::COUNT];  // (entropy-conserving pair: the first line's)
    R M[NP][3];
    fetch_nodes<N>(A.U, stride, e, tid, u);
    if constexpr (FACE) {
#pragma unroll
        for (int q = 0; q < (EC ? 1 : FL); ++q)
#pragma unroll
          for (int h = 0; h < HF; ++h) fetch_face<N, R>(A, stride, pl, e, face_line<N>(wtid - 64 * L::LW, q), h, sn[q][h]);
    } else {
      const LineTask<N> t(wtid);
      if (HF == 1) fetch_face<N, R>(A, stride, pl, e, t, 1, sn[0][1]);
      const R* g = geo_field<R>(A.mesh, stride, 3 * t.d) + static_cast<long long>(e) * NN;
#pragma unroll
      for (int m = 0; m < NP; ++m)
#pragma unroll
        for (int c = 0; c < 3; ++c) M[m][c] = (g + c * stride)[t.end_node(m)];
    }
    if (tid < NP) {
      double w = A.basis.inv_w[0];
#pragma unroll
      for (int i = 1; i < NP; ++i) w = tid == i ? A.basis.inv_w[i] : w;
      sW[tid] = w;
    }
    double p_ref = 0.0, e_ref = 0.0, T_ref = 0.0, beta_ref = 0.0;
    if (MIXED && A.ph.mixed_ref) {
      typedef const __attribute__((address_space(4))) double* Row;  // (scalar loads)
      double s0[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) s0[v] = *(Row)(uintptr_t)(A.U + v * stride + static_cast<long long>(e) * NN);
      const Prim P = primitives(s0, A.ph);
      p_ref = P.p;
      e_ref = EC ? P.p / (A.ph.gm1 * P.rho) : P.e;
      T_ref = P.T;
      beta_ref = 0.5 * P.rho / P.p;
    }
    if (MIXED && tid == 0) {
      sW[NP] = p_ref;
      sW[NP + 1] = e_ref;
      sW[NP + 2] = beta_ref;
      sW[NP + 3] = T_ref;
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const unsigned n = tid + r * BS;
      if (n < NN) {
        const double* s = u[r];
        const double ir = rcp_nr(s[0]);
        const double vx = s[1] * ir, vy = s[2] * ir, vz = s[3] * ir;
        const double q2 = vx * vx + vy * vy + vz * vz;
        const double p = A.ph.gm1 * (s[4] - 0.5 * s[0] * q2);
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
        sF[Fd::TS * EB + l] = static_cast<R>(p * A.ph.inv_R * ir - T_ref);
        if (MIXED && (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N)) {
          double* own = reinterpret_cast<double*>(sF + Fd::OWN) + face_node_index<N>(i, j, k);
#pragma unroll
          for (int v = 0; v < 5; ++v) own[v * Fd::NB] = s[v];
        }
      }
    }
    phase_end();

    // ---- line phase: flux differencing; faces (on the other wave(s)) -----------
    const auto face = [&](const LineTask<N>& t, int h, const double (&s)[FaceReads<R>::COUNT], double (&fs)[5]) {
      R gv[3], gT;
      curv_face<N, R, EC>(again(args), sF, t, h, pl.neighbour(t.d, h) < 0, s, gv, gT, fs);
#pragma unroll
      for (int k = 0; k < 3; ++k) sF[Fd::end_at(t.d, 8 * h + k, t.ab)] = gv[k];
      if constexpr (!MIXED)
#pragma unroll
        for (int k = 0; k < 5; ++k) sF[Fd::end_at(t.d, 8 * h + 3 + k, t.ab)] = fs[k];
      if constexpr (Fd::KEEP_T)
        gt[h] = gT;
      else
        sF[Fd::GT + h * LINES + t.d * NF + t.ab] = gT;
    };
    if constexpr (FACE) {
      const LineArgs& B = again(args);
      const int lane = again(wtid) - 64 * L::LW;
      if constexpr (EC) {
        // one line after the other (the Roe flux is long), the next one's values in
        // flight meanwhile
        const long long st = B.mesh.nE * NN;
        double cur[HF][FaceReads<R>::COUNT], nxt[HF][FaceReads<R>::COUNT], fs[HF][5];
#pragma unroll
        for (int h = 0; h < HF; ++h)
#pragma unroll
          for (int v = 0; v < FaceReads<R>::COUNT; ++v) cur[h][v] = sn[0][h][v];
#pragma unroll 1
        for (int q = 0; q < FL; ++q) {
          const LineTask<N> t = face_line<N>(lane, q), tn = face_line<N>(lane, q + 1 < FL ? q + 1 : q);
          if (FL > 1)
#pragma unroll
            for (int h = 0; h < HF; ++h) fetch_face<N, R>(B, st, pl, e, tn, h, nxt[h]);
#pragma unroll
          for (int h = 0; h < HF; ++h) {
            face(t, h, cur[h], fs[h]);
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (MIXED)
#pragma unroll
            for (int r = 0; r < FL; ++r)
#pragma unroll
              for (int h = 0; h < HF; ++h)
#pragma unroll
                for (int v = 0; v < 5; ++v) fe[r][h][v] = r == q ? fs[h][v] : fe[r][h][v];
          if (FL > 1)
#pragma unroll
            for (int h = 0; h < HF; ++h)
#pragma unroll
              for (int v = 0; v < FaceReads<R>::COUNT; ++v) cur[h][v] = nxt[h][v];
        }
      } else {
#pragma unroll
        for (int q = 0; q < FL; ++q)
#pragma unroll
          for (int h = 0; h < HF; ++h) {
            double fs[5];
            face(face_line<N>(lane, q), h, sn[q][h], fs);
            if constexpr (MIXED)
#pragma unroll
              for (int v = 0; v < 5; ++v) fe[q][h][v] = fs[v];
          }
      }
    } else {
      if constexpr (HF == 1) {
        face(LineTask<N>(again(wtid)), 1, sn[0][1], fe[0][1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      const LineArgs& B = again(args);
      const LineTask<N> t(again(wtid));
#pragma unroll
      for (int m = 0; m < NP; ++m)
#pragma unroll
        for (int c = 0; c < 3; ++c) M[m][c] *= R(0.5);
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int m = 0; m < NP; ++m) acc[v][m] = R(0);
      if constexpr (!EC) {
        curv_pairs<N, R, EC>(B, sF, head, t, M, acc);
      } else {
        // (the means' version from the line's extremes, as in line_device.hpp)
        const R two_ref = MIXED ? static_cast<R>(2.0 * sW[NP + 2]) : R(0);
        R lo[2], hi[2];
#pragma unroll
        for (int m = 0; m < NP; ++m) {
          const R r = sF[t.node(m)], b = sF[4 * EB + t.node(m)];
          lo[0] = m == 0 || r < lo[0] ? r : lo[0];
          hi[0] = m == 0 || r > hi[0] ? r : hi[0];
          lo[1] = m == 0 || b < lo[1] ? b : lo[1];
          hi[1] = m == 0 || b > hi[1] ? b : hi[1];
        }
        const R dr = hi[0] - lo[0], sr = hi[0] + lo[0], db = hi[1] - lo[1], sb = two_ref + (hi[1] + lo[1]);
        const bool mid = dr >= R(0.01) * sr || db >= R(0.01) * sb;
        const bool large = dr >= R(0.1) * sr || db >= R(0.1) * sb;
        const long long st = B.mesh.nE * NN;
        const R* g = geo_field<R>(B.mesh, st, 3 * t.d) + static_cast<long long>(e) * NN;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(large) != 0, 0))
          curv_rows<N, R, 2>(B, sF, head, t, g, st, acc);
        else if (!MIXED && __builtin_amdgcn_ballot_w64(mid) != 0)
          curv_rows<N, R, 1>(B, sF, head, t, g, st, acc);
        else
          curv_pairs<N, R, EC>(B, sF, head, t, M, acc);
      }
      if (MIXED) {  // strong form at the ends: their own flux
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int m = h ? N : 0;
          R x[NQ], f[6];
#pragma unroll
          for (int c = 0; c < NQ; ++c) x[c] = sF[c * EB + t.node(m)];
          curv_pair<N, R, EC, 0>(B.ph, head, x, M[m], x, M[m], f);
#pragma unroll
          for (int v = 0; v < NV; ++v) acc[v][m] += (h ? R(0.5) : R(-0.5)) * f[v];
        }
      }
      settle(acc);
    }
  }
  phase_end();

  // ---- line phase: derivatives of u, v, w (line lanes) and T (face lanes) ------
  double invJ[ROUNDS];
  R Ja[VISC ? ROUNDS : 1][9];  // the nodes' metric terms, in flight meanwhile
  R fn[FACE ? FL : 2][3];      // the neighbours' normal viscous flux at the ends
  {
    const LineArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const unsigned n = node_of<N>(again(tid), r);
      invJ[r] = (A.mesh.geo + 9 * stride + static_cast<long long>(e) * NN)[n];
      if (VISC)
#pragma unroll
        for (int c = 0; c < 9; ++c) Ja[r][c] = (geo_field<R>(A.mesh, stride, c) + static_cast<long long>(e) * NN)[n];
    }
  }
  if constexpr (!FACE) {
    const LineArgs& A = again(args);
    const LineTask<N> t(again(wtid));
    R gh[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (!MIXED)
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v][h ? N : 0] += sF[Fd::end_at(t.d, 8 * h + 3 + v, t.ab)];
#pragma unroll
      for (int c = 0; c < 3; ++c) gh[h][c] = sF[Fd::end_at(t.d, 8 * h + c, t.ab)];
    }
    if (L::UNIFORM) wave_reuse();  // (the ends' values lie in the gradient fields)
    if (VISC) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int nb = pl.neighbour(t.d, h);
        const R* src = static_cast<const R*>(A.ffv) + static_cast<long long>(nb >= 0 ? nb : e) * (6 * 4 * NF) +
                       (2 * t.d + 1 - h) * (4 * NF);
#pragma unroll
        for (int c = 0; c < 3; ++c) fn[h][c] = load_once(&(src + c * NF)[static_cast<unsigned>(t.ab)]);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        R q[NP], g[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) q[m] = sF[(1 + c) * EB + t.node(m)];
        line_derivative<N, R, MIXED>(A.basis, q, gh[0][c], gh[1][c], g);
#pragma unroll
        for (int m = 0; m < NP; ++m) sF[(GS + 3 * c + t.d) * EB + t.node(m)] = g[m];
      }
    }
    settle(acc);
  } else if (VISC) {
    const LineArgs& A = again(args);
    const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
    for (int q = 0; q < FL; ++q) {
      const LineTask<N> t = face_line<N>(lane, q);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int nb = pl.neighbour(t.d, h);
        fn[q][h] = load_once(&(static_cast<const R*>(A.ffv) + static_cast<long long>(nb >= 0 ? nb : e) * (6 * 4 * NF) +
                               ((2 * t.d + 1 - h) * 4 + 3) * NF)[static_cast<unsigned>(t.ab)]);
      }
      R T[NP], g[NP];
#pragma unroll
      for (int m = 0; m < NP; ++m) T[m] = sF[Fd::TS * EB + t.node(m)];
      if constexpr (!Fd::KEEP_T)
#pragma unroll
        for (int h = 0; h < 2; ++h) gt[h] = sF[Fd::GT + h * LINES + t.d * NF + t.ab];
      line_derivative<N, R, MIXED>(A.basis, T, gt[0], gt[1], g);
#pragma unroll
      for (int m = 0; m < NP; ++m) sF[(GS + 9 + t.d) * EB + t.node(m)] = g[m];
    }
  }
  if (VISC) {
    phase_end();

    // ---- node phase: physical gradients -> contravariant half viscous fluxes ----
    {
      const LineArgs& A = again(args);
      const int ts = again(tid);
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        const unsigned n = ts + r * BS;
        if (n < NN) {
          const int i = n % NP, j = (n / NP) % NP, k = n / NF;
          const int l = L::at(i, j, k);
          const R c0 = static_cast<R>(sW[i]), c1 = static_cast<R>(sW[j]), c2 = static_cast<R>(sW[k]);
          const R ij = static_cast<R>(invJ[r]);
          const R(&J)[9] = Ja[r];
          R g[12];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const R h = q < 3 ? ij : R(0.5) * ij;  // (velocities are halves)
            const R g0 = h * c0 * sF[(GS + 3 * q) * EB + l], g1 = h * c1 * sF[(GS + 3 * q + 1) * EB + l],
                    g2 = h * c2 * sF[(GS + 3 * q + 2) * EB + l];
#pragma unroll
            for (int d = 0; d < 3; ++d) g[3 * q + d] = J[d] * g0 + J[3 + d] * g1 + J[6 + d] * g2;
          }
          double rT = 1.0;
          if (A.ph.suth)
            rT = viscosity_ratio(A.ph, static_cast<double>(sF[Fd::TS * EB + l]) + (MIXED ? sW[NP + 3] : 0.0));
          R tau[6], qT[3];
          stress64<R>(g, static_cast<R>(A.ph.mu * rT), static_cast<R>(A.ph.kappa * rT), tau, qT);
          const R u = R(2) * sF[EB + l], v = R(2) * sF[2 * EB + l], w = R(2) * sF[3 * EB + l];
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            R f[4];
            contra_viscous<R>(u, v, w, tau, qT, J[3 * d], J[3 * d + 1], J[3 * d + 2], f);
#pragma unroll
            for (int c = 0; c < 4; ++c) sF[(GS + 3 * c + d) * EB + l] = f[c];
          }
        }
      }
    }
    phase_end();
  }

  // the own state and G of the update are in flight over the rest
  __builtin_amdgcn_sched_barrier(0);
  const int tl = again(tid);
  double gA[ROUNDS][5], u[ROUNDS][5];
  if (RK) {
    const LineArgs& A = again(args);
    const long long stride = A.mesh.nE * NN;
    const double* G = A.st.read_G ? A.out : A.U;  // (the first stage has no G)
    fetch_nodes<N>(A.U, stride, e, tl, u);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int v = 0; v < 5; ++v)
        gA[r][v] = load_once(&(G + v * stride + static_cast<long long>(e) * NN)[node_of<N>(tl, r)]);
  }

  // ---- line phase: derivatives of the viscous fluxes ------------------------
  R fv[3][NP];  // mixed precision: added apart, in FP64
  // (ghosts: half the neighbour's flux; at a wall the own stresses, and the energy flux
  // without their work: f - 2 u . tau)
  if constexpr (VISC && !FACE) {
    const LineArgs& A = again(args);
    const LineTask<N> t(again(wtid));
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      R f[NP], g[NP], gw[2];
#pragma unroll
      for (int m = 0; m < NP; ++m) f[m] = sF[(GS + 3 * c + t.d) * EB + t.node(m)];
#pragma unroll
      for (int h = 0; h < 2; ++h) gw[h] = pl.neighbour(t.d, h) < 0 ? f[h ? N : 0] : R(0.5) * fn[h][c];
      line_derivative<N, R, false>(A.basis, f, gw[0], gw[1], g);
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        if (MIXED)
          fv[c][m] = g[m];
        else
          acc[1 + c][m] -= g[m];
      }
    }
    if (MIXED)
      settle(fv);
    else
      settle(acc);
  } else if constexpr (VISC) {
    const LineArgs& A = again(args);
    const int lane = again(wtid) - 64 * L::LW;
#pragma unroll
    for (int q = 0; q < FL; ++q) {
      const LineTask<N> t = face_line<N>(lane, q);
      R f[NP], gw[2];
#pragma unroll
      for (int m = 0; m < NP; ++m) f[m] = sF[(GS + 9 + t.d) * EB + t.node(m)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int l = t.node(h ? N : 0);
        R w = R(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) w += sF[(1 + c) * EB + l] * sF[(GS + 3 * c + t.d) * EB + l];
        gw[h] = pl.neighbour(t.d, h) < 0 ? f[h ? N : 0] - R(4) * w : R(0.5) * fn[q][h];
      }
      line_derivative<N, R, false>(A.basis, f, gw[0], gw[1], eh[q]);
    }
    settle(eh);
  }

  __builtin_amdgcn_sched_barrier(0);
  // ---- sums of the three directions, scaling, output --------------------------
  phase_end();
  if constexpr (!FACE) {
    const LineTask<N> t(again(wtid));
    R* o = sF + (MIXED ? 4 : 5) * t.d * EB;
    const double p_ref = MIXED ? sW[NP] : 0.0, e_ref = MIXED ? sW[NP + 1] : 0.0;
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int l = t.node(m);
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v * EB + l] = acc[v][m];
      if constexpr (MIXED)
        reinterpret_cast<double*>(sF + (12 + 2 * t.d) * EB)[l] =
            static_cast<double>(acc[4][m]) + e_ref * static_cast<double>(acc[0][m]) + p_ref * static_cast<double>(acc[NV - 1][m]);
      else
        o[4 * EB + l] = acc[4][m];
    }
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
    const double c[3] = {sW[i], sW[j], sW[k]};
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double s = 0.0;
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
        s = d == 0 ? c[0] * f : s + c[d] * f;
      }
      ut[r][v] = s;
    }
  }
  if constexpr (MIXED) {  // the faces' parts, in FP64, and the viscous sums, over the sums just read
    settle(ut);
    phase_end();
    double* sE = reinterpret_cast<double*>(sF);
    R* const sV = sF + 20 * LINES;
    if constexpr (VISC && !FACE) {
      const LineTask<N> t(again(wtid));
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < NP; ++m) sV[(3 * t.d + c) * EB + t.node(m)] = fv[c][m];
    }
    if constexpr (FACE || HF == 1) {
      const int lane = FACE ? again(wtid) - 64 * L::LW : again(wtid);
#pragma unroll
      for (int q = 0; q < FF; ++q) {
        const LineTask<N> t = FACE ? face_line<N>(lane, q) : LineTask<N>(lane);
#pragma unroll
        for (int h = H0; h < H1; ++h)
#pragma unroll
          for (int v = 0; v < 5; ++v) sE[(5 * h + v) * LINES + t.d * NF + t.ab] = fe[q][h][v];
      }
    }
    phase_end();
    const double iw = sW[0];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const unsigned n = node_of<N>(tl, r);
      const int i = n % NP, j = (n / NP) % NP, k = n / NF;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int x = d == 0 ? i : (d == 1 ? j : k);
        if (x == 0 || x == N) {
          const int ab = d == 0 ? j + NP * k : (d == 1 ? i + NP * k : i + NP * j);
          const double* o = sE + (x == N ? 5 : 0) * LINES + d * NF + ab;
#pragma unroll
          for (int v = 0; v < 5; ++v) ut[r][v] += iw * o[v * LINES];
        }
        if (VISC)
#pragma unroll
          for (int c = 0; c < 3; ++c) ut[r][1 + c] -= sW[x] * static_cast<double>(sV[(3 * d + c) * EB + L::at(i, j, k)]);
      }
    }
  }
  const LineArgs& A = again(args);
  const long long stride = A.mesh.nE * NN, base = static_cast<long long>(e) * NN;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const unsigned n = again(tid) + r * BS;
    if (NN % BS == 0 || n < NN) {
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double x = -2.0 * invJ[r] * ut[r][v];
        if (RK) {
          const double g = A.st.read_G ? A.st.A * gA[r][v] + A.st.dt * x : A.st.dt * x;
          store_once(&(A.out + v * stride + base)[n], g);
          store_once(&(A.U_out + v * stride + base)[n], u[r][v] + A.st.B * g);
        } else {
          store_once(&(A.out + v * stride + base)[n], x);
        }
      }
    }
  }
}

template <int N, typename R, bool RK, bool VISC, bool EC>
__global__ __launch_bounds__(Line<N>::BS) __attribute__((amdgpu_waves_per_eu(CurvFields<N, R, EC>::WAVES))) void k_rhs_curv(
    LineArgs) {
  using L = Line<N>;
  extern __shared__ double lds[];
  const LineArgsPtr args = (LineArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int tid = threadIdx.x, blk = static_cast<int>(blockIdx.x);
  const int e = xcd_remap(blk, gridDim.x);
  // (which wave takes the faces: line_device.hpp)
  const int turn = L::UNIFORM ? ((blk >> 3) + (blk >> 8)) & 3 : 0;
  const int wtid = L::UNIFORM ? (tid + 64 * turn) & 255 : tid;
  if (__builtin_amdgcn_readfirstlane(wtid) >= 64 * L::LW)
    curv_phases<N, R, RK, VISC, EC, true>(args, lds, e, tid, wtid);
  else
    curv_phases<N, R, RK, VISC, EC, false>(args, lds, e, tid, wtid);
}

template <int N, typename R, bool EC, bool RK>
hipError_t curv_line_n(const LineArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.mesh.nE)), block(Line<N>::BS);
  const size_t lds = CurvFields<N, R, EC>::BYTES;
  if (a.ph.viscous)
    hipLaunchKernelGGL((k_rhs_curv<N, R, RK, true, EC>), grid, block, lds, s, a);
  else
    hipLaunchKernelGGL((k_rhs_curv<N, R, RK, false, EC>), grid, block, lds, s, a);
  return hipGetLastError();
}

template <typename R, bool EC>
hipError_t curv_line_dispatch(int N, bool rk, const LineArgs& a, hipStream_t s) {
  switch (N) {
    case 3: return rk ? curv_line_n<3, R, EC, true>(a, s) : curv_line_n<3, R, EC, false>(a, s);
    case 5: return rk ? curv_line_n<5, R, EC, true>(a, s) : curv_line_n<5, R, EC, false>(a, s);
    case 7: return rk ? curv_line_n<7, R, EC, true>(a, s) : curv_line_n<7, R, EC, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace dg
