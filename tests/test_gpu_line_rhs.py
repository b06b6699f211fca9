"""The line-lane right-hand side (GPU) at the sizes where its work split can go
wrong: fewer elements than XCDs, element counts that are no multiple of the
XCDs, every degree, walls of both kinds on each axis, with and without
viscosity, Sutherland's law, the right-hand side alone and as an RK step.

With the entropy-conserving pair also states of smaller spreads, where a line's
logarithmic means all take their long or their short series (the default states
take the third path).

Criterion: per conserved variable, relative L2 error against the FP64 oracle on the
same seeded state, <= 1e-12 (FP64); in mixed precision <= 1e-4, an FP32 evaluation's
6e-8 amplified by the cancellation of pair fluxes in a derivative and the factor
between the terms' and their sum's size.
"""

import numpy as np
import pytest
import torch

from oracle.dgsem import rhs, rk_step
from oracle.mesh import Mesh
from oracle.physics import Gas
from paper_2606_18927_amd import dgsem

from _cases import random_faces, random_state
from _gpu import need_gpu, rel_l2, say, to_dev

pytestmark = pytest.mark.gpu
P = "periodic"
BOUND = {"fp64": 1e-12, "mixed": 1e-4}


@pytest.mark.parametrize("N,n,bc,opts", [
    (7, (1, 1, 1), (P, P, P), {}),
    (7, (3, 1, 3), ("wall", P, "wallmodel"), {"suth": True}),
    (7, (9, 8, 8), (P, "wall", P), {}),
    (7, (3, 3, 1), (P, P, "wall"), {"viscous": False}),
    (5, (1, 1, 1), (P, P, P), {}),
    (5, (3, 3, 2), ("wallmodel", "wall", P), {"suth": True}),
    (5, (2, 3, 3), (P, "wall", "wall"), {"viscous": False, "central": True}),
    (3, (1, 1, 1), ("wall", P, P), {}),
    (3, (5, 3, 7), (P, "wallmodel", "wall"), {"suth": True}),
    (3, (9, 1, 2), (P, P, P), {"viscous": False}),
])
@pytest.mark.parametrize("flux,precision,spread", [
    ("kg_llf", "fp64", 0.2), ("ec_roe", "fp64", 0.2), ("ec_roe", "fp64", 0.02), ("ec_roe", "fp64", 0.002),
    ("kg_llf", "mixed", 0.2), ("ec_roe", "mixed", 0.2), ("ec_roe", "mixed", 0.02)])
def test_rhs_and_rk_step(N, n, bc, opts, flux, precision, spread):
    need_gpu()
    say("case", N, n, bc, opts, flux, precision, spread)
    rng = np.random.default_rng(100 * N + n[0])
    faces = tuple(random_faces(n[d], 0.0, 1.0 + d, rng) for d in range(3))
    mesh = Mesh(N, faces, bc=bc, T_wall=1.1, wm_node=2)
    suth = (1.0, 0.4) if opts.get("suth") else None
    g = Gas(gamma=1.4, R=1.0 / (1.4 * 0.01), mu=0.01, Pr=0.72, sutherland=suth is not None, T_ref=1.0, S=0.4)
    U = random_state(mesh, g.gamma, g.R, rng, vel_amp=1.0, p_mean=g.R, p_amp=min(0.05, spread),
                     rho_amp=spread)
    kw = {"viscous": opts.get("viscous", True), "central_only": opts.get("central", False), "flux": flux}
    S = dgsem.Solver(dgsem.MeshSpec(N, faces, bc, 1.1, 2), g.gamma, g.R, g.mu, g.Pr, precision=precision,
                     sutherland=suth, **kw)
    Ud = to_dev(U.numpy())
    ref = rhs(U, mesh, g, **kw).numpy()
    e = rel_l2(S.eval_rhs(Ud).cpu().numpy(), ref)
    say("rhs", e)
    assert np.all(e < BOUND[precision])
    # three steps: the increment, so that every stage (with and without G) counts
    dt = 1e-3 / max(np.abs(ref[v]).max() / np.abs(U[v].numpy()).max() for v in range(5))
    S.set_state(Ud)
    S.rk_step(dt, 3)
    S.sync()
    want = rk_step(U, mesh, g, dt, 3, **kw).numpy() - U.numpy()
    got = S.get_state().cpu().numpy().reshape(want.shape) - U.numpy()
    # the increment is a difference of states: their rounding, eps |U| / |dU|, is
    # part of it
    tol = BOUND[precision] + 4 * 2.3e-16 * np.array(
        [np.linalg.norm(U[v].numpy()) / np.linalg.norm(want[v]) for v in range(5)])
    e = rel_l2(got, want)
    say("rk", e, tol)
    assert np.all(e < tol)


@pytest.mark.parametrize("N,n,bc,opts", [
    (7, (2, 3, 1), (P, "wall", P), {"suth": True}),
    (5, (1, 2, 3), ("wall", P, "wall"), {}),
    (5, (3, 1, 2), (P, P, "wall"), {"viscous": False}),
    (3, (3, 2, 5), (P, "wall", P), {"central": True}),
])
@pytest.mark.parametrize("flux,spread", [("kg_llf", 0.2), ("ec_roe", 0.2), ("ec_roe", 0.02), ("ec_roe", 0.002)])
def test_rhs_vjp(N, n, bc, opts, flux, spread):
    """The vector-Jacobian product with line lanes against the oracle's reverse mode,
    per variable relative L2 <= 1e-11."""
    from oracle.adjoint import rhs_vjp
    need_gpu()
    say("vjp case", N, n, bc, opts, flux, spread)
    rng = np.random.default_rng(7 * N + n[0])
    faces = tuple(random_faces(n[d], 0.0, 1.0 + d, rng) for d in range(3))
    mesh = Mesh(N, faces, bc=bc, T_wall=1.1)
    suth = (1.0, 0.4) if opts.get("suth") else None
    g = Gas(gamma=1.4, R=1.0 / (1.4 * 0.01), mu=0.01, Pr=0.72, sutherland=suth is not None, T_ref=1.0, S=0.4)
    U = random_state(mesh, g.gamma, g.R, rng, vel_amp=1.0, p_mean=g.R, p_amp=min(0.05, spread), rho_amp=spread)
    lam = torch.tensor(rng.standard_normal(tuple(U.shape)))
    kw = {"viscous": opts.get("viscous", True), "central_only": opts.get("central", False), "flux": flux}
    S = dgsem.Solver(dgsem.MeshSpec(N, faces, bc, 1.1), g.gamma, g.R, g.mu, g.Pr, with_adjoint=True,
                     sutherland=suth, **kw)
    got = S.eval_rhs_vjp(to_dev(U.numpy()), to_dev(lam.numpy())).cpu().numpy()
    S.sync()
    e = rel_l2(got, rhs_vjp(U, lam, mesh, g, **kw).numpy())
    say("vjp", e)
    assert np.all(e < 1e-11)


@pytest.mark.parametrize("N,n,opts", [
    (3, (1, 1, 1), {}),
    (3, (3, 1, 2), {"suth": True}),
    (5, (1, 3, 2), {}),
    (7, (2, 1, 3), {"suth": True}),
    (7, (1, 2, 1), {"viscous": False, "central": True}),
])
@pytest.mark.parametrize("flux,precision,spread", [
    ("kg_llf", "fp64", 0.2), ("ec_roe", "fp64", 0.2), ("ec_roe", "fp64", 0.02), ("ec_roe", "fp64", 0.002),
    ("kg_llf", "mixed", 0.2), ("ec_roe", "mixed", 0.2), ("ec_roe", "mixed", 0.02)])
def test_curved_rhs(N, n, opts, flux, precision, spread):
    """The right-hand side on warped elements, same criteria."""
    from oracle import curvilinear as cv
    from paper_2606_18927_amd import workloads
    need_gpu()
    say("curved case", N, n, opts, flux, precision, spread)
    X = workloads.warped_nodes(dgsem.lgl(N)[0], n, amp=0.05)
    mesh = cv.CurvMesh(N, torch.as_tensor(X))
    suth = (1.0, 0.4) if opts.get("suth") else None
    g = Gas(gamma=1.4, R=1.0, mu=0.02, Pr=0.72, sutherland=suth is not None, T_ref=1.0, S=0.4)
    U = random_state(mesh, g.gamma, g.R, np.random.default_rng(60 + N), p_amp=spread, rho_amp=spread)
    kw = {"viscous": opts.get("viscous", True), "central_only": opts.get("central", False), "flux": flux}
    S = dgsem.Solver(dgsem.MeshSpec(N, None, (P, P, P), 1.0, nodes=X), g.gamma, g.R, g.mu, g.Pr, precision=precision,
                     sutherland=suth, **kw)
    got = S.eval_rhs(to_dev(U.numpy())).cpu().numpy()
    S.sync()
    e = rel_l2(got, cv.rhs(U, mesh, g, **kw).numpy())
    say("curved rhs", e)
    assert np.all(e < BOUND[precision])


def test_reverse_step_in_place():
    """The reverse step may write its cotangent over the one it reads or over the
    stage states: the same result as into a buffer of its own."""
    need_gpu()
    N, n = 3, (2, 3, 2)
    rng = np.random.default_rng(5)
    faces = tuple(random_faces(n[d], 0.0, 1.0 + d, rng) for d in range(3))
    mesh = Mesh(N, faces, bc=(P, P, P))
    g = Gas(gamma=1.4, R=1.0, mu=0.01, Pr=0.72)
    U = to_dev(random_state(mesh, g.gamma, g.R, rng).numpy()).reshape(-1)
    S = dgsem.Solver(dgsem.MeshSpec(N, faces, (P, P, P)), g.gamma, g.R, g.mu, g.Pr, with_adjoint=True)
    lam = to_dev(rng.standard_normal(U.numel()))
    stages = S.rk_record_stages(U, 1e-3, 1)
    want = S.rk_step_vjp_stages(stages[0], 1e-3, lam, out=torch.empty_like(lam)).clone()
    same = lam.clone()
    S.rk_step_vjp_stages(stages[0], 1e-3, same, out=same)
    for s in (0, 2, 4):
        st = stages.clone()
        S.rk_step_vjp_stages(st[0], 1e-3, lam, out=st[0][s])
        S.sync()
        assert torch.equal(st[0][s], want)
    S.sync()
    assert torch.equal(same, want)


@pytest.mark.parametrize("N,n,wavy,opts", [
    (3, (3, 1, 2), False, {"suth": True}),
    (3, (2, 2, 2), True, {}),
    (5, (1, 3, 2), False, {}),
    (5, (2, 2, 1), True, {"suth": True}),
    (5, (2, 1, 2), False, {"viscous": False}),
    (7, (2, 1, 3), False, {}),
    (7, (1, 2, 2), True, {"suth": True}),
    (7, (1, 2, 1), False, {"viscous": False, "central": True}),
])
@pytest.mark.parametrize("flux,precision,spread", [
    ("kg_llf", "fp64", 0.2), ("ec_roe", "fp64", 0.2), ("ec_roe", "fp64", 0.02), ("ec_roe", "fp64", 0.002),
    ("kg_llf", "mixed", 0.2), ("ec_roe", "mixed", 0.2), ("ec_roe", "mixed", 0.02)])
def test_curved_rk_steps(N, n, wavy, opts, flux, precision, spread):
    """Three RK steps on warped elements and between wavy walls, as in test_rhs_and_rk_step:
    the increment against the oracle's, with the states' rounding in the bound."""
    from oracle import curvilinear as cv
    from paper_2606_18927_amd import workloads
    need_gpu()
    say("curved rk case", N, n, wavy, opts, flux, precision, spread)
    make = workloads.wavy_channel_nodes if wavy else workloads.warped_nodes
    X, bc = make(dgsem.lgl(N)[0], n, amp=0.05), (P, "wall", P) if wavy else (P, P, P)
    mesh = cv.CurvMesh(N, torch.as_tensor(X), bc=bc, T_wall=1.1)
    suth = (1.0, 0.4) if opts.get("suth") else None
    g = Gas(gamma=1.4, R=1.0, mu=0.02, Pr=0.72, sutherland=suth is not None, T_ref=1.0, S=0.4)
    U = random_state(mesh, g.gamma, g.R, np.random.default_rng(80 + N), p_amp=spread, rho_amp=spread)
    kw = {"viscous": opts.get("viscous", True), "central_only": opts.get("central", False), "flux": flux}
    ref = cv.rhs(U, mesh, g, **kw).numpy()
    dt = 1e-3 / max(np.abs(ref[v]).max() / np.abs(U[v].numpy()).max() for v in range(5))
    S = dgsem.Solver(dgsem.MeshSpec(N, None, bc, 1.1, nodes=X), g.gamma, g.R, g.mu, g.Pr, precision=precision,
                     sutherland=suth, **kw)
    S.set_state(to_dev(U.numpy()))
    S.rk_step(dt, 3)
    S.sync()
    want = cv.rk_step(U, mesh, g, dt, 3, **kw).numpy() - U.numpy()
    got = S.get_state().cpu().numpy().reshape(want.shape) - U.numpy()
    tol = BOUND[precision] + 4 * 2.3e-16 * np.array(
        [np.linalg.norm(U[v].numpy()) / np.linalg.norm(want[v]) for v in range(5)])
    e = rel_l2(got, want)
    say("curved rk", e, tol)
    assert np.all(e < tol)


@pytest.mark.parametrize("kind", ["fp64", "mixed", "ec_roe", "curved", "curved_mixed", "graph"])
def test_set_state_after_a_run_that_broke_down(kind):
    """The RK register of an earlier run, here NaN, does not enter the steps after set_state:
    its first stage does not read it.  Bitwise the state of a fresh solver."""
    from paper_2606_18927_amd import workloads
    need_gpu()
    N, n = 5, (2, 1, 2)
    curved = kind.startswith("curved")
    faces = tuple(np.linspace(0.0, 1.0 + d, n[d] + 1) for d in range(3))
    X = workloads.warped_nodes(dgsem.lgl(N)[0], n, amp=0.05) if curved else None
    spec = dgsem.MeshSpec(N, None if curved else faces, (P, P, P), 1.0, nodes=X)
    kw = {"precision": "mixed" if kind.endswith("mixed") else "fp64", "flux": "ec_roe" if kind == "ec_roe" else "kg_llf"}
    U = to_dev(random_state(Mesh(N, faces), 1.4, 1.0, np.random.default_rng(9)).numpy())

    def steps(S):
        S.set_state(U)
        if kind == "graph":
            S.rk_graph_build(1e-4, 2)
            S.rk_graph_launch(1)
        else:
            S.rk_step(1e-4, 2)
        S.sync()
        return S.get_state()

    S = dgsem.Solver(spec, 1.4, 1.0, 0.01, 0.72, **kw)
    S.set_state(torch.full_like(U, float("nan")))
    S.rk_step(1e-4, 1)
    with pytest.raises(dgsem.DgsemError):
        S.sync()
    got = steps(S)
    assert torch.isfinite(got).all()
    assert torch.equal(got, steps(dgsem.Solver(spec, 1.4, 1.0, 0.01, 0.72, **kw)))
