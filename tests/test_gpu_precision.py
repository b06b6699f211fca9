"""Rounding error of the right-hand side (GPU) against the operator in 80-bit floats.

Criterion, FP64: per conserved variable at most 1.5 times the error of a plain FP64
evaluation of the same formulas on the same input (tests/_extended.py in float64),
since the kernels differ from it in the order of their sums only.  The adjoint: the same
against the oracle's FP64 reverse mode (with nodes, weights and derivative matrix rounded
from 80 bits), exact being complex steps of the 80-bit operator.
"""

import numpy as np
import pytest

from paper_2606_18927_amd import dgsem, workloads

from _extended import Operator, box_nodes, lgl
from _gpu import need_gpu, say, state, to_dev

pytestmark = pytest.mark.gpu
P = "periodic"
GAMMA, MU, PR = 1.4, 1.0 / 160.0, 0.72
R = 1.0 / (GAMMA * 0.01)  # Ma = 0.1: p = 71 beside velocities of 1
SIZES = {3: (4, 3, 5), 5: (3, 4, 3), 7: (3, 2, 3)}


def vortex(X):
    """Taylor-Green vortex with noise in velocity and temperature."""
    rng = np.random.default_rng(1)
    noise = lambda: rng.uniform(-1, 1, X.shape[1:])  # noqa: E731
    x, y, z = X
    v = [np.sin(x) * np.cos(y) * np.cos(z) + 0.01 * noise(), -np.cos(x) * np.sin(y) * np.cos(z) + 0.01 * noise(),
         0.01 * noise()]
    p = R + (np.cos(2 * x) + np.cos(2 * y)) * (np.cos(2 * z) + 2) / 16
    rho = p / (R * (1 + 0.002 * noise()))
    return np.stack([rho, *(rho * q for q in v), p / (GAMMA - 1) + 0.5 * rho * sum(q * q for q in v)])


def errors(N, flux, curved):
    """Per variable: the kernel's error, and that of the plain FP64 evaluation."""
    n = SIZES[N]
    faces = tuple(2 * np.pi * np.arange(k + 1) / k for k in n)
    nodes = workloads.warped_nodes(dgsem.lgl(N)[0], n, amp=0.05) if curved else box_nodes(N, faces)
    U = vortex(np.asarray(nodes, dtype=np.float64).reshape(3, n[2], n[1], n[0], N + 1, N + 1, N + 1))
    args = (N, np.asarray(nodes).reshape((3,) + U.shape[1:]), GAMMA, R, MU, PR, flux)
    exact, plain = Operator(*args).rhs(U), Operator(*args, dtype=np.float64).rhs(U)
    S = dgsem.Solver(dgsem.MeshSpec(N, None if curved else faces, (P, P, P), 1.0, nodes=nodes if curved else None),
                     GAMMA, R, MU, PR, flux=flux)
    got = S.eval_rhs(to_dev(U)).cpu().numpy().reshape(U.shape)
    S.sync()
    off = lambda q: np.sqrt(((q - exact) ** 2).reshape(5, -1).sum(1) / (exact ** 2).reshape(5, -1).sum(1)).astype(float)  # noqa: E731
    return off(got), off(plain)


@pytest.mark.parametrize("N", [3, 5, 7])
def test_entropy_conserving_pair(N):
    """With p = rho rcp(2 beta), two roundings more than a division, the Roe flux's pressure
    jumps put 1.7 times this error into mass and energy."""
    need_gpu()
    say("precision case", N)
    e, plain = errors(N, "ec_roe", False)
    say(e, plain, e / plain)
    assert np.all(e <= 1.5 * plain)


@pytest.mark.parametrize("N", [3, 5, 7])
@pytest.mark.parametrize("flux", ["kg_llf", "ec_roe"])
def test_curved_elements(N, flux):
    """The two elements of a face compute its metric vector with different rounding.  Where
    the own flux and the surface flux take different ones, the pressure multiplies the
    difference: 5, 17 and 21 times this error in the momentum (N = 3, 5, 7).  (The
    Kennedy-Gruber energy, from e = E / rho, is left out: 4 times at N = 3.)"""
    need_gpu()
    say("precision case, curved", N, flux)
    e, plain = errors(N, flux, True)
    say(e, plain, e / plain)
    k = 5 if flux == "ec_roe" else 4
    assert np.all(e[:k] <= 1.5 * plain[:k])


# ------------------------------------------------------------- mixed precision

@pytest.mark.parametrize("N", [3, 5, 7])
def test_mixed_uniform_flow(N):
    """In a uniform flow whose fluxes are powers of two every product of the FP32 sums is
    exact, and the coefficients' rows sum to zero exactly: the right-hand side is zero."""
    need_gpu()
    say("uniform flow", N)
    n = SIZES[N]
    faces = tuple(np.cumsum(np.concatenate([[0.0], 0.5 + np.arange(k) / k])) for k in n)
    U = np.empty((5, n[2], n[1], n[0], N + 1, N + 1, N + 1))
    U[:4] = np.array([1.0, 1.0, -0.5, 0.25]).reshape(4, 1, 1, 1, 1, 1, 1)
    U[4] = R / (GAMMA - 1) + 0.5 * (1.0 + 0.25 + 0.0625)
    S = dgsem.Solver(dgsem.MeshSpec(N, faces, (P, P, P), 1.0), GAMMA, R, MU, PR, precision="mixed")
    got = S.eval_rhs(to_dev(U)).cpu().numpy()
    S.sync()
    assert np.all(got == 0.0), np.abs(got).max()


def test_mixed_run_keeps_mass():
    """4000 steps of an inviscid channel flow, N = 5, 8^3 elements.  Each of the N (N + 1)
    additions of a line's mass sum (values below 1) rounds by at most 2^-25, with no
    preferred sign: a standard deviation of 2^-25 sqrt(N (N + 1) / 3) for the line, and of the
    sums over lines and steps by adding variances.  Four of them are allowed; a mean
    error of the sums would grow with the number of steps instead of its root."""
    need_gpu()
    N, n, steps = 5, 8, 4000
    x, w = dgsem.lgl(N)
    faces = [np.linspace(0, 2 * np.pi, n + 1), np.linspace(-1, 1, n + 1), np.linspace(0, np.pi, n + 1)]
    y = 0.5 * (faces[1][:-1, None] + faces[1][1:, None]) + 0.5 * np.diff(faces[1])[:, None] * x
    shape = (n, n, n, N + 1, N + 1, N + 1)
    prof = np.broadcast_to((1.5 * (1 - y * y)).reshape(1, n, 1, 1, N + 1, 1), shape)
    rng = np.random.default_rng(3)
    v = [prof + 0.05 * rng.uniform(-1, 1, shape)] + [0.05 * rng.uniform(-1, 1, shape) for _ in range(2)]
    U = np.stack([np.ones(shape), *v, R / (GAMMA - 1) + 0.5 * sum(q * q for q in v)])
    dt = 0.1 / (2 * N + 1) / (11 * n / 2)
    S = dgsem.Solver(dgsem.MeshSpec(N, tuple(faces), (P, "wall", P), 1.0), GAMMA, R, 0.0, PR, precision="mixed",
                     viscous=False)
    S.set_state(to_dev(U))
    S.rk_step(dt, steps)
    S.sync()
    W = w[:, None, None] * w[None, :, None] * w[None, None, :] / 8 / n ** 3  # of the volume
    drift = abs(((S.get_state().cpu().numpy().reshape(U.shape)[0] - 1.0) * W).sum())
    line = 2.0 ** -25 * np.sqrt(N * (N + 1) / 3)
    s = [2 * n / (f[-1] - f[0]) for f in faces]
    rate = np.sqrt(sum((w ** 2).sum() ** 2 * n ** 3 * (2 * sd * line / 8 / n ** 3) ** 2 for sd in s))
    bound = 4 * rate * dt * np.sqrt(steps)
    say("mass drift", drift, "bound", bound)
    assert drift < bound


def test_mixed_channel_energy_after_500_steps():
    """The kinetic energy of the 48x32x48 channel after 500 steps, mixed against FP64.
    With the sums' rounding errors free of a mean it is 6e-12 off; a mean error of 3e-10 of
    the flux made it 1.6e-10."""
    need_gpu()
    wl = workloads.WORKLOADS["channel_n5_48x32x48"]
    U, dt = state(wl)
    J = {}
    for prec in ("fp64", "mixed"):
        S = dgsem.solver_for(wl, precision=prec)
        S.set_state(to_dev(U))
        S.rk_step(dt, 500)
        S.sync()
        J[prec] = S.kinetic_energy(S.get_state()).item()
        say(prec, J[prec])
        del S
    e = abs(J["mixed"] - J["fp64"]) / J["fp64"]
    say("J", e)
    assert e < 4e-11


def vjp_errors(flux, variables, monkeypatch):
    """Per given variable, N = 5, 8 elements, 40 % noise: the kernel's VJP error at 40 random nodes
    relative to their rms, and that of the oracle's reverse mode."""
    import torch
    import oracle.dgsem
    from oracle.adjoint import rhs_vjp
    from oracle.mesh import Mesh
    from oracle.physics import Gas
    N = 5
    rounded = lambda a: torch.as_tensor(a.astype(np.float64))  # noqa: E731
    monkeypatch.setattr(oracle.dgsem, "lgl", lambda n: tuple(rounded(a) for a in lgl(n)[:2]))
    monkeypatch.setattr(oracle.dgsem, "diff_matrix", lambda n: rounded(lgl(n)[2]))
    faces = (2 * np.pi * np.array([0, 0.45, 1]),) * 3
    rng = np.random.default_rng(5)
    shape = (2, 2, 2, N + 1, N + 1, N + 1)
    noise = lambda a: rng.uniform(-a, a, shape)  # noqa: E731
    rho, p, v = 1 + noise(0.4), R * (1 + noise(0.2)), [a + noise(0.5) for a in (0.3, -0.2, 0)]
    U = np.stack([rho, *(rho * q for q in v), p / (GAMMA - 1) + 0.5 * rho * sum(q * q for q in v)])
    lam = rng.uniform(-1, 1, U.shape) * np.array([1, 1, 1, 1, 0.01]).reshape(5, 1, 1, 1, 1, 1, 1)
    op = Operator(N, box_nodes(N, faces), GAMMA, R, MU, PR, flux, dtype=np.clongdouble)
    at = rng.choice(rho.size, 40, replace=False)
    exact = np.empty((len(variables), at.size), dtype=np.longdouble)
    for r, v in enumerate(variables):
        for k, q in enumerate(at):
            W = U.astype(np.clongdouble)
            W[v].reshape(-1)[q] += 1j * np.longdouble(1e-30)
            exact[r, k] = (lam * op.rhs(W).imag).sum() / np.longdouble(1e-30)
        say("complex steps of variable", v)
    S = dgsem.Solver(dgsem.MeshSpec(N, faces, (P, P, P), 1.0), GAMMA, R, MU, PR, flux=flux, with_adjoint=True)
    got = S.eval_rhs_vjp(to_dev(U), to_dev(lam)).cpu().numpy().reshape(5, -1)
    S.sync()
    plain = rhs_vjp(torch.as_tensor(U), torch.as_tensor(lam), Mesh(N, faces), Gas(gamma=GAMMA, R=R, mu=MU, Pr=PR),
                    flux=flux).numpy().reshape(5, -1)
    off = lambda q: np.sqrt(((q[variables][:, at] - exact) ** 2).sum(1) / (exact ** 2).sum(1)).astype(float)  # noqa: E731
    return off(got), off(plain)


def test_adjoint_kennedy_gruber(monkeypatch):
    """With the dissipation's cotangents taken through (rho, e), and e formed
    again from rho e, the density's cotangent had 2.5 times this error."""
    need_gpu()
    say("precision case adjoint, Kennedy-Gruber")
    e, plain = vjp_errors("kg_llf", [0, 1, 2, 3, 4], monkeypatch)
    say(e, plain, e / plain)
    assert np.all(e <= 1.5 * plain)


def test_adjoint_entropy_conserving(monkeypatch):
    """Larger jumps: with Q = w D rounded thrice the energy's cotangent had 1.8 times this
    error.  (The others' sits at the face nodes, behind the Roe flux, in a few outliers.)"""
    need_gpu()
    say("precision case adjoint, entropy-conserving")
    e, plain = vjp_errors("ec_roe", [4], monkeypatch)
    say(e, plain, e / plain)
    assert np.all(e <= 1.5 * plain)
