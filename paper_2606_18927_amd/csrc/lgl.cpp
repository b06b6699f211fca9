// Host construction of the Legendre-Gauss-Lobatto basis (paper Sec. 2.2:
// collocation on LGL nodes).
//
// Nodes: -1, +1 and the roots of P_N', found by Newton's method on P_N' with
// the second derivative from Legendre's equation
//   (1 - x^2) P_N'' = 2 x P_N' - N (N+1) P_N,
// started from the Chebyshev-Gauss-Lobatto points -cos(pi j / N).
// Weights: w_j = 2 / (N (N+1) P_N(x_j)^2).
// Derivative matrix: barycentric form D_im = (b_m / b_i) / (x_i - x_m) with
// b_i = 1 / prod_{m != i} (x_i - x_m), and the diagonal by the negative-sum
// rule D_ii = -sum_{m != i} D_im, which makes rows of D annihilate constants
// to rounding.
#include <cmath>
#include <vector>

#include "dg_internal.hpp"

namespace dg {

namespace {

// P_N(x) and P_N'(x) by the three-term recurrence.
void legendre(int N, double x, double& P, double& dP) {
  double p0 = 1.0, p1 = x, d0 = 0.0, d1 = 1.0;
  if (N == 0) {
    P = 1.0;
    dP = 0.0;
    return;
  }
  for (int k = 1; k < N; ++k) {
    const double p2 = ((2.0 * k + 1.0) * x * p1 - k * p0) / (k + 1.0);
    const double d2 = d0 + (2.0 * k + 1.0) * p1;
    p0 = p1;
    p1 = p2;
    d0 = d1;
    d1 = d2;
  }
  P = p1;
  dP = d1;
}

}  // namespace

void lgl_nodes_weights(int N, std::vector<double>& xi, std::vector<double>& w) {
  xi.assign(N + 1, 0.0);
  w.assign(N + 1, 0.0);
  xi[0] = -1.0;
  xi[N] = 1.0;
  const double nn1 = N * (N + 1.0);
  for (int j = 1; j < N; ++j) {
    double x = -std::cos(M_PI * j / N);
    for (int it = 0; it < 100; ++it) {
      double P, dP;
      legendre(N, x, P, dP);
      const double d2P = (2.0 * x * dP - nn1 * P) / (1.0 - x * x);
      const double dx = dP / d2P;
      x -= dx;
      if (std::fabs(dx) < 1e-16 * (1.0 + std::fabs(x))) break;
    }
    xi[j] = x;
  }
  // exact symmetry of the rule
  for (int j = 0; j <= N / 2; ++j) {
    const double a = 0.5 * (xi[N - j] - xi[j]);
    xi[j] = -a;
    xi[N - j] = a;
  }
  if (N % 2 == 0) xi[N / 2] = 0.0;
  for (int j = 0; j <= N; ++j) {
    double P, dP;
    legendre(N, xi[j], P, dP);
    w[j] = 2.0 / (nn1 * P * P);
  }
}

void lgl_diff_matrix(const std::vector<double>& xi, std::vector<double>& D) {
  const int NP = static_cast<int>(xi.size());
  std::vector<double> b(NP, 1.0);
  for (int i = 0; i < NP; ++i) {
    double prod = 1.0;
    for (int m = 0; m < NP; ++m)
      if (m != i) prod *= (xi[i] - xi[m]);
    b[i] = 1.0 / prod;
  }
  D.assign(NP * NP, 0.0);
  for (int i = 0; i < NP; ++i) {
    double diag = 0.0;
    for (int m = 0; m < NP; ++m) {
      if (m == i) continue;
      const double v = (b[m] / b[i]) / (xi[i] - xi[m]);
      D[i * NP + m] = v;
      diag -= v;
    }
    D[i * NP + i] = diag;
  }
}

// Q_im = w_i D_im = 2 / (N (N + 1) P_N(x_i) P_N(x_m) (x_i - x_m)) for i != m, from
// nodes refined in extended precision, so that the rounded values keep the
// exact antisymmetry.
//
// The FP32 entries: rounded one by one, a row with its end value (-+1/2) sums to 3e-7 after
// division by the end weight (N = 5), a systematic gradient of that times the mean
// velocity, and a linear profile's slope is off by 2e-7 (N = 7).  So they are multiples of
// 2^-27 (of their own last place where that is coarser) near Q, at most 8e-8 away, such
// that the rows sum to zero exactly, a constant has no derivative, and their first, then
// second and third moments are off least (the slope by 6e-8, at N = 7 by 1e-8): an integer
// programme solved once for each N.
void lgl_line_basis(int N, DevBasis& b) {
  const int NP = N + 1;
  const long double nn1 = static_cast<long double>(N) * (N + 1);
  std::vector<long double> x(NP), P(NP);
  std::vector<double> xi, w;
  lgl_nodes_weights(N, xi, w);
  const auto legendre_ld = [N](long double t, long double& p, long double& dp) {
    long double p0 = 1.0L, d0 = 0.0L;
    p = t;
    dp = 1.0L;
    for (int k = 1; k < N; ++k) {
      const long double p2 = ((2 * k + 1) * t * p - k * p0) / (k + 1), d2 = d0 + (2 * k + 1) * p;
      p0 = p;
      p = p2;
      d0 = dp;
      dp = d2;
    }
  };
  for (int j = 0; j < NP; ++j) {
    long double t = xi[j], p, dp;
    for (int it = 0; it < 3 && j > 0 && j < N; ++it) {
      legendre_ld(t, p, dp);
      t -= dp * (1.0L - t * t) / (2.0L * t * dp - nn1 * p);
    }
    x[j] = t;
  }
  for (int j = 0; j <= N / 2; ++j) {
    const long double a = 0.5L * (x[N - j] - x[j]);
    x[j] = -a;
    x[N - j] = a;
  }
  for (int j = 0; j < NP; ++j) {
    long double dp;
    legendre_ld(x[j], P[j], dp);
    b.inv_w[j] = static_cast<double>(nn1 * P[j] * P[j] / 2.0L);
  }
  static const int kUnits3[4] = {90487016, -34562960, 11184808, 125049976};
  static const int kUnits5[9] = {90743856, -36115196, 20085100, -12078820, 4473924, 128185160, -58561424, 33198940, 130546288};
  static const int kUnits7[16] = {90777192,  -36283312, 20601980,  -13470616, 9307326,   -6220450,  2396744,  128493680,
                                  -59729596, 36601196,  -24588206, 16220568,  131654728, -62852596, 38689116, 132249128};
  const int* const units = N == 3 ? kUnits3 : (N == 5 ? kUnits5 : kUnits7);
  for (int i = 0; i <= N / 2; ++i)
    for (int m = i + 1; m <= N - i; ++m) {
      const long double q = 2.0L / (nn1 * P[i] * P[m] * (x[i] - x[m]));
      const int k = i * N - i * (i - 1) + m - i - 1;
      b.Q[k] = static_cast<double>(q);
      b.Qf[k] = std::ldexp(static_cast<float>(units[k]), -27);
    }
}

}  // namespace dg
