"""The line kernels' coefficients Q = diag(w) D (CPU, from the built library): the FP64
entries against 80-bit floats, and the FP32 entries' exact row sums."""

import ctypes
from fractions import Fraction

import numpy as np
import pytest

from paper_2606_18927_amd import dgsem

from _extended import lgl


class Basis(ctypes.Structure):  # dg::DevBasis
    _fields_ = [("D", ctypes.c_void_p), ("inv_w_end", ctypes.c_double), ("Q", ctypes.c_double * 16),
                ("Qf", ctypes.c_float * 16), ("inv_w", ctypes.c_double * 8)]


def full(N, packed):
    """The (N+1)^2 matrix of the packed entries: antisymmetric, Q_{N-m,N-i} = Q_im."""
    Q = [[None] * (N + 1) for _ in range(N + 1)]
    for i in range(N + 1):
        for m in range(N + 1):
            a, b = min(i, m), max(i, m)
            if a + b > N:
                a, b = N - b, N - a
            if i == m:
                Q[i][m] = Fraction(-1, 2) if i == 0 else Fraction(1, 2) if i == N else Fraction(0)
            else:
                Q[i][m] = (1 if i < m else -1) * Fraction(packed[a * N - a * (a - 1) + b - a - 1])
    return Q


@pytest.mark.parametrize("N", [3, 5, 7])
def test_line_coefficients(N):
    b = Basis()
    dgsem.lib()._ZN2dg14lgl_line_basisEiRNS_8DevBasisE(N, ctypes.byref(b))
    x, w, D = lgl(N)
    ref = w[:, None] * D
    for packed, tol in ((b.Q, 2.0 ** -53), (b.Qf, 8e-8)):
        got = np.array(full(N, packed), dtype=np.longdouble)
        off = ~np.eye(N + 1, dtype=bool)
        assert np.all(abs(got - ref)[off] <= tol)
    # FP32: the rows sum to zero exactly, and differentiate x to better than 1e-7
    Q = full(N, b.Qf)
    assert all(sum(row) == 0 for row in Q)
    slope = (np.array(Q, dtype=np.longdouble) @ x) / w
    assert np.all(abs(slope - 1) < 1e-7)
