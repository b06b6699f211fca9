"""The operator in 80-bit floats (numpy), for tests of the rounding error of the
FP64 and mixed-precision kernels.

Periodic boxes, Navier-Stokes with constant viscosity, either flux pair, written in
the curvilinear form throughout (an axis-aligned box is the curved mesh whose nodes
lie on it).  The formulas are those of ``oracle.dgsem`` and ``oracle.curvilinear``;
the sums run over node arrays (nz, ny, nx, k, j, i).
"""

import numpy as np

LD = np.longdouble


def mag(x):
    """|x|, continued to complex steps as sign(Re x) x."""
    return x * np.sign(x.real)


def lgl(N):
    """Nodes, weights and derivative matrix (rows summing to zero)."""
    leg = np.polynomial.legendre
    P = np.zeros(N + 1, dtype=LD)
    P[N] = 1
    d1 = leg.legder(P)
    d2 = leg.legder(d1)
    x = np.sort(leg.legroots(leg.legder(P.astype(float))).real).astype(LD)
    for _ in range(4):
        x = x - leg.legval(x, d1) / leg.legval(x, d2)
    x = np.concatenate([[LD(-1)], x, [LD(1)]])
    x = (x - x[::-1]) / 2
    PN = leg.legval(x, P)
    D = np.zeros((N + 1, N + 1), dtype=LD)
    for i in range(N + 1):
        for m in range(N + 1):
            if m != i:
                D[i, m] = PN[i] / PN[m] / (x[i] - x[m])
        D[i, i] = -D[i].sum()
    return x, 2 / (N * (N + 1) * PN * PN), D


def box_nodes(N, faces):
    """Node coordinates (3, nz, ny, nx, k, j, i) of an axis-aligned box."""
    x = lgl(N)[0]
    t = []
    for f in faces:
        f = np.asarray(f).astype(LD)
        t.append((f[:-1, None] + f[1:, None]) / 2 + np.diff(f)[:, None] / 2 * x)
    NP, n = N + 1, [a.shape[0] for a in t]
    shape = (n[2], n[1], n[0], NP, NP, NP)
    return np.stack([np.broadcast_to(t[0].reshape(1, 1, -1, 1, 1, NP), shape),
                     np.broadcast_to(t[1].reshape(1, -1, 1, 1, NP, 1), shape),
                     np.broadcast_to(t[2].reshape(-1, 1, 1, NP, 1, 1), shape)])


class Operator:
    """dtype: the type everything is computed in (float64: what a plain evaluation of
    the same formulas is off by; clongdouble: with complex steps)."""

    def __init__(self, N, nodes, gamma, R, mu, Pr, flux, dtype=LD):
        self.N, self.ec, self.dtype = N, flux == "ec_roe", dtype
        self.gamma, self.R, self.mu = dtype(gamma), dtype(R), dtype(mu)
        self.kappa = self.mu * self.gamma * self.R / ((self.gamma - 1) * dtype(Pr))
        _, w, D = lgl(N)
        self.D, self.w0 = D.astype(dtype), dtype(w[0])
        X = [x - x[..., :1, :1, :1] for x in np.asarray(nodes).astype(dtype)]
        dX = [[self.diff(X[n], d) for d in range(3)] for n in range(3)]
        J = sum(dX[0][a] * (dX[1][b] * dX[2][c] - dX[1][c] * dX[2][b]) for a, b, c in ((0, 1, 2), (1, 2, 0), (2, 0, 1)))
        self.Ja = [[None] * 3 for _ in range(3)]
        for n in range(3):
            m, l = (n + 1) % 3, (n + 2) % 3
            V = [X[l] * dX[m][d] - X[m] * dX[l][d] for d in range(3)]
            for i in range(3):
                a, b = (i + 1) % 3, (i + 2) % 3
                self.Ja[i][n] = -(self.diff(V[b], a) - self.diff(V[a], b)) / 2
        self.inv_J = 1 / J

    def diff(self, q, d):
        return np.moveaxis(np.tensordot(self.D, q, axes=(1, 5 - d)), 0, 5 - d)

    def two_point(self, a, b, M):
        """Flux of states (rho, u, v, w, p, E) contracted with the metric vector M."""
        v = [(a[k] + b[k]) / 2 for k in (1, 2, 3)]
        un = sum(x * m for x, m in zip(v, M))
        if not self.ec:
            mass, p = (a[0] + b[0]) / 2 * un, (a[4] + b[4]) / 2
            e = (a[5] / a[0] + b[5] / b[0]) / 2
            return [mass] + [mass * x + p * m for x, m in zip(v, M)] + [mass * e + p * un]
        ba, bb = a[0] / (2 * a[4]), b[0] / (2 * b[4])
        mass, p = self.ln_mean(a[0], b[0]) * un, (a[0] + b[0]) / 2 / (ba + bb)
        q2 = sum(a[k] ** 2 + b[k] ** 2 for k in (1, 2, 3)) / 2
        f = [mass] + [mass * x + p * m for x, m in zip(v, M)]
        return f + [mass * (1 / (2 * (self.gamma - 1) * self.ln_mean(ba, bb)) - q2 / 2)
                    + f[1] * v[0] + f[2] * v[1] + f[3] * v[2]]

    def ln_mean(self, a, b):
        f = (a - b) / (a + b)
        u = f * f
        F = u / 21
        for k in range(19, 1, -2):  # atanh f / f for f^2 below 1e-2 (first dropped term 1e-22 / 23)
            F = u * (F + 1 / self.dtype(k))
        F = 1 + F
        near = u < 1e-2
        fs = np.where(near, self.dtype(0.5), f)
        return (a + b) / (2 * np.where(near, F, np.arctanh(fs) / fs))

    def surface(self, L, Rt, M):
        f = self.two_point(L, Rt, M)
        size = np.sqrt(sum(m * m for m in M))
        n = [m / size for m in M]
        cons = lambda q: [q[0], q[0] * q[1], q[0] * q[2], q[0] * q[3], q[5]]  # noqa: E731
        c = [np.sqrt(self.gamma * q[4] / q[0]) for q in (L, Rt)]
        un = [sum(q[1 + k] * n[k] for k in range(3)) for q in (L, Rt)]
        if not self.ec:
            lam = np.maximum(mag(un[0]) + c[0], mag(un[1]) + c[1])
            return [x - size * lam / 2 * (r - l) for x, l, r in zip(f, cons(L), cons(Rt))]
        sl, sr = np.sqrt(L[0]), np.sqrt(Rt[0])
        wl, wr = sl / (sl + sr), sr / (sl + sr)
        v = [wl * L[1 + k] + wr * Rt[1 + k] for k in range(3)]
        H = wl * (L[5] + L[4]) / L[0] + wr * (Rt[5] + Rt[4]) / Rt[0]
        q2 = sum(x * x for x in v)
        a2 = (self.gamma - 1) * (H - q2 / 2)
        a, rho = np.sqrt(a2), sl * sr
        u = sum(x * y for x, y in zip(v, n))
        dv = [Rt[1 + k] - L[1 + k] for k in range(3)]
        du, dp = sum(x * y for x, y in zip(dv, n)), Rt[4] - L[4]

        def hh(lam, l, r):
            d = np.maximum(np.maximum(lam - l, r - lam), 0)
            return np.where(mag(lam) < d, (lam * lam + d * d) / np.where(d > 0, 2 * d, 1), mag(lam))

        t1 = hh(u - a, un[0] - c[0], un[1] - c[1]) * (dp - rho * a * du) / (2 * a2)
        t5 = hh(u + a, un[0] + c[0], un[1] + c[1]) * (dp + rho * a * du) / (2 * a2)
        t2, ts = mag(u) * (Rt[0] - L[0] - dp / a2), mag(u) * rho
        sh = [dv[k] - du * n[k] for k in range(3)]
        dis = [t1 + t2 + t5] + [(t1 + t2 + t5) * v[k] + (t5 - t1) * a * n[k] + ts * sh[k] for k in range(3)]
        dis += [t1 * (H - u * a) + t2 * q2 / 2 + t5 * (H + u * a) + ts * sum(x * y for x, y in zip(v, sh))]
        return [x - size / 2 * y for x, y in zip(f, dis)]

    def rhs(self, U):
        N = self.N
        U = np.asarray(U).astype(self.dtype)
        rho, v = U[0], [U[k] / U[0] for k in (1, 2, 3)]
        p = (self.gamma - 1) * (U[4] - rho / 2 * sum(x * x for x in v))
        P = [rho, *v, p, U[4]]
        line = lambda q, d: np.moveaxis(q, 5 - d, 0)  # noqa: E731
        grad = []
        for q in [*v, p / (rho * self.R)]:
            ref = []
            for d in range(3):
                g, lo, hi = self.diff(q, d), line(q, d)[0], line(q, d)[N]
                s = (hi + np.roll(lo, -1, 2 - d)) / 2
                line(g, d)[N] += (s - hi) / self.w0
                line(g, d)[0] -= (np.roll(s, 1, 2 - d) - lo) / self.w0
                ref.append(g)
            grad.append([sum(self.Ja[r][n] * ref[r] for r in range(3)) * self.inv_J for n in range(3)])
        div = grad[0][0] + grad[1][1] + grad[2][2]
        tau = [[self.mu * (grad[a][b] + grad[b][a] - (2 * div / 3 if a == b else 0)) for b in range(3)] for a in range(3)]
        out = np.zeros_like(U)
        for d in range(3):
            M = self.Ja[d]
            fv = [sum(tau[a][b] * M[b] for b in range(3)) for a in range(3)]
            fv.append(sum(v[a] * fv[a] for a in range(3)) + self.kappa * sum(grad[3][b] * M[b] for b in range(3)))
            L = [line(q, d) for q in P]
            ML = [line(m, d) for m in M]
            acc = np.zeros((5,) + L[0].shape, dtype=self.dtype)
            for i in range(N + 1):
                for m in range(i, N + 1):
                    f = self.two_point([q[i] for q in L], [q[m] for q in L], [(x[i] + x[m]) / 2 for x in ML])
                    for k in range(5):
                        acc[k][i] += 2 * self.D[i, m] * f[k]
                        if m != i:
                            acc[k][m] += 2 * self.D[m, i] * f[k]
            roll = lambda x, s: np.roll(x, s, 2 - d)  # noqa: E731
            F = self.surface([q[N] for q in L], [roll(q[0], -1) for q in L], [x[N] for x in ML])
            for k in range(4):
                F[1 + k] = F[1 + k] - (line(fv[k], d)[N] + roll(line(fv[k], d)[0], -1)) / 2
            for e, s in ((N, 1), (0, -1)):
                m = [x[N] if e else roll(x[N], 1) for x in ML]  # the face's one normal, on both sides
                un = sum(L[1 + n][e] * m[n] for n in range(3))
                own = [L[0][e] * un] + [L[0][e] * un * L[1 + n][e] + L[4][e] * m[n] for n in range(3)] + [(L[5][e] + L[4][e]) * un]
                for k in range(5):
                    o = own[k] - (line(fv[k - 1], d)[e] if k else 0)
                    acc[k][e] += s * ((F[k] if e else roll(F[k], 1)) - o) / self.w0
            for k in range(5):
                r = np.moveaxis(acc[k], 0, 5 - d)
                out[k] -= r - (self.diff(fv[k - 1], d) if k else 0)
        return out * self.inv_J
