"""Multigrid transfers and stencil kernels at the shapes where their split can
go wrong: axes that end on an odd fine node, one-cell axes, levels on both
sides of the size at which the nine-wave stencil kernel takes over, and rows
that cross the 64-node groups of the restriction.

A preconditioner only changes how fast CG gets there, so an error in it shows
as a lost iteration count or as no convergence.  The bound on the iterations
is the Jacobi count divided by 2 on the small meshes (the multigrid parity
tests ask 5x on theirs); the solution is checked against the oracle's
residual, which a solve to rtol 1e-10 meets to 2e-10 (its own FP64 residual
plus rounding of the same size)."""
import numpy as np
import pytest

import oracle
import paper_2603_07038_amd as etm
import workloads as W

pytestmark = pytest.mark.gpu


def _solve(prob, th, precision, **opt):
    plan = etm.Plan(prob, prob.sample_J_half(etm.cfl_dt(prob), 4), precision=precision, n_steps=4, history=False, **opt)
    plan.write(etm.ETM_FIELD_THETA, th)
    plan.mech_solve()
    return plan, plan.sync()


@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("shape", [(33, 31, 9), (64, 5, 1), (1, 40, 37), (3, 2, 70), (65, 33, 8), (40, 41, 2)])
def test_odd_and_thin_meshes_converge_as_fast(shape, precision):
    prob = W.random_problem(11 + sum(shape), *shape, n_steps=4, R=2, n_ports=1, void_top=0,
                            mech_bc=W.MECH_CLAMP_ZMIN)
    prob.cg_rtol = 1e-10
    th = np.random.default_rng(3).uniform(0.0, 40.0, (prob.nz + 1, prob.ny + 1, prob.nx + 1))
    plan, info = _solve(prob, th, precision, mg_coarse_dofs=60)
    assert info["mg_levels"] >= 3 and info["cg_relres"] <= prob.cg_rtol
    jac = _solve(prob, th, precision, mech_precond=etm.ETM_PRECOND_JACOBI)[1]
    assert info["cg_iters"] <= jac["cg_iters"] / 2
    o = oracle.Oracle(prob)
    f = o.mech_rhs(th, o.mech_mask())
    res = f - o.mech_apply(o.mech_mask(), plan.u())
    assert np.linalg.norm(res) <= 2e-10 * np.linalg.norm(f)


# level 1 has 95 x 95 x 12 = 108,300 nodes (one thread per node) or 95 x 95 x 10
# = 90,250 (nine waves per 64); level 2 takes the nine-wave kernel in both
@pytest.mark.parametrize("nz", [22, 18])
def test_both_stencil_kernels_precondition_alike(nz):
    prob = W.package(188, 188, nz, 5, n_bits=4, max_traces=4)
    prob.cg_rtol = 1e-10
    z, y, x = np.meshgrid(np.linspace(0, 1, nz + 1), np.linspace(0, 1, 189), np.linspace(0, 1, 189), indexing="ij")
    th = 20.0 + 10.0 * np.sin(5 * x + 3 * y) * np.cos(4 * y - z)
    its = []
    for precision in (etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED):
        plan, info = _solve(prob, th, precision)
        assert info["cg_relres"] <= prob.cg_rtol
        its.append(info["cg_iters"])
        o = oracle.Oracle(prob)
        f = o.mech_rhs(th, o.mech_mask())
        res = f - o.mech_apply(o.mech_mask(), plan.u())
        assert np.linalg.norm(res) <= 2e-10 * np.linalg.norm(f)
    # refinement restarts cost the mixed path a few iterations, no more
    assert its[1] <= its[0] + 16 and max(its) <= 60


# smoothing degrees: a step that reads no direction, one that takes x for it, and
# (from 3 on) ones that read and store it, with the three vectors of a level
# changing places; both preconditioners are symmetric, so CG gets there
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("degree", [(1, 1), (2, 1), (3, 2), (4, 3), (1, 4)])
def test_every_smoothing_degree_converges(degree, precision):
    prob = W.random_problem(58, 40, 33, 9, n_steps=4, R=2, n_ports=1, void_top=0, mech_bc=W.MECH_CLAMP_ZMIN)
    prob.cg_rtol = 1e-10
    th = np.random.default_rng(3).uniform(0.0, 40.0, (prob.nz + 1, prob.ny + 1, prob.nx + 1))
    plan, info = _solve(prob, th, precision, mg_coarse_dofs=60, mg_degree=degree)
    assert info["mg_levels"] >= 3 and info["cg_relres"] <= prob.cg_rtol
    jac = _solve(prob, th, precision, mech_precond=etm.ETM_PRECOND_JACOBI)[1]
    assert info["cg_iters"] <= jac["cg_iters"] / 2
    o = oracle.Oracle(prob)
    f = o.mech_rhs(th, o.mech_mask())
    res = f - o.mech_apply(o.mech_mask(), plan.u())
    assert np.linalg.norm(res) <= 2e-10 * np.linalg.norm(f)
