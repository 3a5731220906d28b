"""The matrix-free HEX8 operator at the edges of its tiles (31 x 7 owned nodes)
and of its z-chunks, both precisions, against the oracle's solve.

Tolerance: both sides solve to a relative residual of 1e-12 (the oracle to
1e-13); as in the parity tests the displacement and the stress of such solves
agree to 1e-8 of their largest value."""
import numpy as np
import pytest

import oracle
import paper_2603_07038_amd as etm
import workloads as W

pytestmark = pytest.mark.gpu


def rel_err(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


# nodes per axis: one tile exactly, one more, two tiles; one, two and many
# planes; a column long enough for several chunks
@pytest.mark.parametrize("shape", [(30, 6, 1), (31, 7, 2), (61, 13, 5), (62, 14, 4), (1, 1, 1), (7, 3, 190),
                                   (33, 20, 17)])
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
def test_solve_at_tile_edges_matches_oracle(shape, precision):
    prob = W.random_problem(77 + sum(shape), *shape, n_steps=4, R=2, n_ports=1,
                            void_top=1 if shape[2] > 2 else 0, mech_bc=W.MECH_CLAMP_ZMIN)
    prob.cg_rtol = 1e-12
    o = oracle.Oracle(prob)
    dt = o.cfl_dt()
    plan = etm.Plan(prob, prob.sample_J_half(dt, 4), dt=dt, precision=precision, n_steps=4, history=False)
    rng = np.random.default_rng(5)
    th = rng.uniform(0.0, 40.0, (prob.nz + 1, prob.ny + 1, prob.nx + 1))
    plan.write(etm.ETM_FIELD_THETA, th)
    plan.mech_solve()
    info = plan.sync()
    assert info["cg_relres"] <= prob.cg_rtol
    q, _, _ = o.mech_solve(th, o.mech_mask(), rtol=1e-13)
    q = np.asarray(q).reshape(plan.u().shape)
    assert rel_err(plan.u(), q) < 1e-8
    vm = o.von_mises(th, q)
    vm = vm[0] if isinstance(vm, tuple) else vm
    assert rel_err(plan.read(etm.ETM_FIELD_VM), np.asarray(vm).reshape(prob.mat.shape)) < 1e-8


# A long strip of one cell layer: the operator's 2118 blocks are more than the
# 2052 blocks of 64 x 4 nodes, and each writes a row of partials.
def test_solve_with_more_tiles_than_node_blocks_matches_oracle():
    prob = W.random_problem(9, 32800, 7, 1, n_steps=4, R=2, n_ports=1, void_top=0, mech_bc=W.MECH_CLAMP_ZMIN)
    prob.cg_rtol = 1e-12
    o = oracle.Oracle(prob)
    th = np.random.default_rng(5).uniform(0.0, 40.0, (prob.nz + 1, prob.ny + 1, prob.nx + 1))
    q, _, _ = o.mech_solve(th, o.mech_mask(), rtol=1e-13)
    dt = o.cfl_dt()
    for precision in (etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED):
        print("precision", precision, flush=True)
        plan = etm.Plan(prob, prob.sample_J_half(dt, 4), dt=dt, precision=precision, n_steps=4, history=False)
        plan.write(etm.ETM_FIELD_THETA, th)
        plan.mech_solve()
        info = plan.sync()
        assert info["cg_relres"] <= prob.cg_rtol
        assert rel_err(plan.u(), np.asarray(q).reshape(plan.u().shape)) < 1e-8
