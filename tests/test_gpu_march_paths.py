"""The march's port records and its choice of z-chunk, at the sizes where they
can go wrong.

Tolerances: several sources on one port edge are summed in the order they are
given, as the oracle sums them, so the bars are those of the parity tests
(FP64 1e-9 of the field's max norm; mixed e 1e-5, temperature 1e-6).  The
z-chunk only splits the work: every split gives the same bits."""
import json

import numpy as np
import pytest

import oracle
import paper_2603_07038_amd as etm
import workloads as W

pytestmark = pytest.mark.gpu


def rel_err(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("n_ports", [1, 160])
def test_ports_in_every_direction_and_shared_edges(precision, n_ports):
    prob = W.random_problem(41, 5, 4, 3, n_steps=24, R=3, n_ports=n_ports, amp=3e10, em_bc=(0,) * 6)
    o = oracle.Oracle(prob)
    dt = o.cfl_dt()
    J = prob.sample_J_half(dt, 24)
    if n_ports > 1:
        edge = list(zip(prob.port_dir, prob.port_i, prob.port_j, prob.port_k))
        assert len(set(edge)) < len(edge) and set(prob.port_dir) == {0, 1, 2}
    plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=24, history=False)
    plan.advance(24)
    plan.sync()
    st, _ = o.run(dt, 24, J, stride=0, probes=None)
    scale = max(np.abs(x).max() for x in st["e"])
    e_bar, t_bar = (1e-9, 1e-9) if precision == etm.ETM_PREC_FP64 else (1e-5, 1e-6)
    for g, w in zip(plan.e(), st["e"]):
        assert np.abs(g - w).max() <= e_bar * scale
    assert rel_err(plan.read(etm.ETM_FIELD_THETA), st["theta"]) <= t_bar


# one generation of blocks at chunks of 1, 2, 3 and 4 planes, and the first
# sizes past it (mixed | FP64 tiles differ)
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("shape", [(61, 61, 38), (80, 77, 48), (110, 100, 40), (131, 118, 43), (152, 120, 43),
                                   (190, 131, 44)])
def test_chunk_choice_does_not_change_results(shape, precision):
    prob = W.random_problem(sum(shape), *shape, n_steps=12, R=6, n_ports=6, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 12)
    out = []
    for slabs in (0, 2):  # slabs keep the chunk of a shared launch
        plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=12, history=False, em_slabs=slabs)
        plan.advance(12)
        plan.sync()
        out.append(plan.e() + plan.e_prev() + [plan.read(etm.ETM_FIELD_THETA)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][0]).max() > 0


# the edges of the FP64 tile (32 x 8 nodes), and launches either side of the
# size from which their one-time data bypasses the caches (2.37 M nodes); a
# launch of slabs never does
@pytest.mark.parametrize("shape", [(30, 6, 5), (31, 7, 5), (32, 8, 5), (33, 16, 6), (158, 150, 97), (160, 152, 98)])
def test_fp64_tiles_and_streaming_do_not_change_results(shape):
    prob = W.random_problem(sum(shape), *shape, n_steps=8, R=4, n_ports=6, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    out = []
    for slabs in (0, 2):
        plan = etm.Plan(prob, J, dt=dt, precision=etm.ETM_PREC_FP64, n_steps=8, history=False, em_slabs=slabs)
        plan.advance(8)
        plan.sync()
        out.append(plan.e() + plan.e_prev() + [plan.read(etm.ETM_FIELD_THETA)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][0]).max() > 0
    if shape[0] < 100:
        st, _ = oracle.Oracle(prob).run(dt, 8, J, stride=0, probes=None)
        scale = max(np.abs(x).max() for x in st["e"])
        for g, w in zip(out[0][:3], st["e"]):
            assert np.abs(g - w).max() <= 1e-9 * scale


def test_fp64_batch_above_the_streaming_size_matches_solo():
    probs = [W.random_problem(q, 120 + q, 110, 45, n_steps=8, R=4, n_ports=4, amp=3e10) for q in range(4)]
    assert sum((p.nx + 1) * (p.ny + 1) * (p.nz + 1) for p in probs) * 113 > 1 << 28
    plans = []
    for _ in range(2):
        plans.append([etm.Plan(p, p.sample_J_half(etm.cfl_dt(p), 8), precision=etm.ETM_PREC_FP64, n_steps=8,
                               history=False) for p in probs])
    batch = etm.Batch(4)
    for p in plans[0]:
        batch.attach(p)
    batch.advance(8)
    for a, b in zip(*plans):
        a.sync()
        b.advance(8)
        b.sync()
        for x, y in zip(a.e() + a.e_prev(), b.e() + b.e_prev()):
            np.testing.assert_array_equal(x, y)


# The mixed march's two forms give the same bits: the edges of the tile (64 x 4
# nodes), chunks of one to four planes, and launches either side of the size
# from which a plan takes the tiles (3.16 M nodes; the last two, the second of
# which pads its plane by more than 30 % and keeps the runs).
@pytest.mark.parametrize("kchunk", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", [(4, 3, 3), (62, 3, 4), (63, 4, 5), (64, 5, 6), (65, 7, 7), (127, 8, 9)])
def test_mixed_tiles_match_runs(shape, kchunk):
    prob = W.random_problem(sum(shape), *shape, n_steps=9, R=4, n_ports=min(6, shape[0]), amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 9)
    cls = str(int(np.floor(np.log2(max(shape[0] * shape[1] * shape[2], 1)))))
    out = []
    for layout in (None, 1, 2):
        plan = etm.Plan(prob, J, dt=dt, precision=etm.ETM_PREC_MIXED, n_steps=9, history=False)
        if layout is None:
            plan.advance(9)
        else:
            batch = etm.Batch(1, json.dumps({"kchunk": {cls: kchunk}, "layout": {cls: layout}}))
            batch.attach(plan)
            batch.advance(9)
        plan.sync()
        out.append(plan.e() + [plan.read(etm.ETM_FIELD_THETA)])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("shape", [(254, 190, 64), (255, 195, 64), (129, 190, 150)])
def test_mixed_streaming_plans_match_runs(shape):
    prob = W.random_problem(sum(shape), *shape, n_steps=8, R=4, n_ports=6, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    cls = str(int(np.floor(np.log2(shape[0] * shape[1] * shape[2]))))
    out = []
    for form in ("solo", "slabs", "runs"):
        plan = etm.Plan(prob, J, dt=dt, precision=etm.ETM_PREC_MIXED, n_steps=8, history=False,
                        em_slabs=2 if form == "slabs" else 0)
        if form == "runs":
            batch = etm.Batch(1, json.dumps({"layout": {cls: 1}}))
            batch.attach(plan)
            batch.advance(8)
        else:
            plan.advance(8)
        plan.sync()
        out.append(plan.e() + [plan.read(etm.ETM_FIELD_THETA)])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][0]).max() > 0


# The thermal kernel over chunks of 1 and 4 planes (64 x 4 columns, the last
# chunk short), one thermal block per EM step so that every step adds pending
# Joule power, against the oracle.
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("shape", [(5, 4, 3), (63, 3, 5), (64, 5, 4), (66, 180, 30)])
def test_thermal_columns(shape, precision):
    prob = W.random_problem(sum(shape), *shape, n_steps=4, R=1, n_ports=4, amp=3e10)
    o = oracle.Oracle(prob)
    dt = o.cfl_dt()
    J = prob.sample_J_half(dt, 4)
    plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=4, history=False)
    plan.advance(4)
    plan.sync()
    st, _ = o.run(dt, 4, J, stride=0, probes=None)
    assert rel_err(plan.read(etm.ETM_FIELD_THETA), st["theta"]) <= (1e-9 if precision == etm.ETM_PREC_FP64 else 1e-6)


# The refresh after a temperature change skips planes and blocks without a
# temperature-dependent conductor; the full one at a restore does not: a march
# that goes on from its own checkpoint is bitwise the uninterrupted one.  The
# second shape refreshes chunks of two planes.
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("shape", [(40, 30, 12), (258, 250, 40)])
def test_coefficient_refresh_matches_full(shape, precision):
    prob = W.random_problem(sum(shape), *shape, n_steps=8, R=2, n_ports=4, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=8, history=False)
    plan.advance(4)
    plan.sync()
    again = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=8, history=False)
    again.restore(plan.checkpoint())
    out = []
    for p in (plan, again):
        p.advance(4)
        p.sync()
        out.append(p.e() + [p.read(etm.ETM_FIELD_THETA)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][3]).max() > 0


# FP64 meshes of few rows of nodes take tiles of 64 x 4 (above 256 blocks): the
# tile's edges, one to nine rows, and a launch whose one-time data bypasses the
# caches; slabs, and a batch together with a mesh of 32 x 8 tiles.
@pytest.mark.parametrize("shape", [(62, 1, 150), (63, 3, 140), (64, 2, 140), (127, 8, 40), (129, 3, 70), (2000, 3, 300)])
def test_fp64_flat_tiles_do_not_change_results(shape):
    prob = W.random_problem(sum(shape), *shape, n_steps=8, R=4, n_ports=6, amp=3e10, em_bc=(1, 0, 0, 0, 1, 0))
    other = W.random_problem(7, 33, 20, 12, n_steps=8, R=4, n_ports=4, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    out = []
    for form in ("solo", "slabs", "batch"):
        plan = etm.Plan(prob, J, dt=dt, precision=etm.ETM_PREC_FP64, n_steps=8, history=False,
                        em_slabs=2 if form == "slabs" else 0)
        if form == "batch":
            second = etm.Plan(other, other.sample_J_half(etm.cfl_dt(other), 8), precision=etm.ETM_PREC_FP64, n_steps=8,
                              history=False)
            batch = etm.Batch(2)
            batch.attach(plan)
            batch.attach(second)
            batch.advance(8)
            alone = etm.Plan(other, other.sample_J_half(etm.cfl_dt(other), 8), precision=etm.ETM_PREC_FP64, n_steps=8,
                             history=False)
            alone.advance(8)
            for a, b in zip(alone.e(), second.e()):
                np.testing.assert_array_equal(a, b)
        else:
            plan.advance(8)
        plan.sync()
        out.append(plan.e() + plan.e_prev() + [plan.read(etm.ETM_FIELD_THETA)])
    for form in out[1:]:
        for a, b in zip(out[0], form):
            np.testing.assert_array_equal(a, b)
    assert max(np.abs(x).max() for x in out[0][:3]) > 0
    st, _ = oracle.Oracle(prob).run(dt, 8, J, stride=0, probes=None)
    scale = max(np.abs(x).max() for x in st["e"])
    for g, w in zip(out[0][:3], st["e"]):
        assert np.abs(g - w).max() <= 1e-9 * scale
    assert rel_err(out[0][6], st["theta"]) <= 1e-9


# A mixed plan just below the size from which it takes the tiles, just above, and
# above it with a plane that tiles pad by more than 30 % (runs): as it is, in
# runs and in tiles (forced through a batch's table).
@pytest.mark.parametrize("shape", [(254, 188, 64), (254, 189, 64), (129, 190, 150)])
def test_mixed_plans_either_side_of_the_streaming_size(shape):
    prob = W.random_problem(sum(shape), *shape, n_steps=8, R=4, n_ports=6, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    cls = str(int(np.floor(np.log2(shape[0] * shape[1] * shape[2]))))
    out = []
    for layout in (None, 1, 2):
        plan = etm.Plan(prob, J, dt=dt, precision=etm.ETM_PREC_MIXED, n_steps=8, history=False)
        if layout:
            batch = etm.Batch(1, json.dumps({"layout": {cls: layout}}))
            batch.attach(plan)
            batch.advance(8)
        else:
            plan.advance(8)
        plan.sync()
        out.append(plan.e() + [plan.read(etm.ETM_FIELD_THETA)])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][0]).max() > 0


# A mixed batch whose nodes stream, in tiles of odd chunks and as the default
# table has it, with a variant that streams by itself and small ones.
@pytest.mark.parametrize("table", ["tiles", "default"])
def test_mixed_batch_above_the_streaming_size_matches_solo(table):
    shapes = [(131, 118, 45), (70, 9, 33), (260, 190, 66), (121, 120, 50), (64, 64, 40), (63, 3, 17)]
    probs = [W.random_problem(q, *s, n_steps=8, R=4, n_ports=4, amp=3e10) for q, s in enumerate(shapes)]
    assert sum((p.nx + 1) * (p.ny + 1) * (p.nz + 1) for p in probs) * 85 > 1 << 28
    plans = []
    for _ in range(2):
        plans.append([etm.Plan(p, p.sample_J_half(etm.cfl_dt(p), 8), precision=etm.ETM_PREC_MIXED, n_steps=8,
                               history=False) for p in probs])
    classes = {int(np.floor(np.log2(p.n_cells))) for p in probs}
    tune = {"kchunk": {str(c): [3, 5, 7][c % 3] for c in classes}, "layout": {str(c): 2 for c in classes}}
    batch = etm.Batch(len(probs), json.dumps(tune) if table == "tiles" else None)
    for p in plans[0]:
        batch.attach(p)
    batch.advance(8)
    for a, b in zip(*plans):
        a.sync()
        b.advance(8)
        b.sync()
        for x, y in zip(a.e() + a.e_prev() + [a.read(etm.ETM_FIELD_THETA)],
                        b.e() + b.e_prev() + [b.read(etm.ETM_FIELD_THETA)]):
            np.testing.assert_array_equal(x, y)


# The thermal kernel over chunks of 8 and of 12 planes (700 blocks or more),
# against the oracle, as in test_thermal_columns.
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
@pytest.mark.parametrize("shape", [(127, 255, 47), (126, 253, 65)])
def test_thermal_long_chunks(shape, precision):
    prob = W.random_problem(sum(shape), *shape, n_steps=3, R=1, n_ports=4, amp=3e10)
    o = oracle.Oracle(prob)
    dt = o.cfl_dt()
    J = prob.sample_J_half(dt, 3)
    plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=3, history=False)
    plan.advance(3)
    plan.sync()
    st, _ = o.run(dt, 3, J, stride=0, probes=None)
    assert rel_err(plan.read(etm.ETM_FIELD_THETA), st["theta"]) <= (1e-9 if precision == etm.ETM_PREC_FP64 else 1e-6)


# The refresh over chunks of 8 planes (4800 blocks or more), the last one short,
# against the full one at a restore, as in test_coefficient_refresh_matches_full.
@pytest.mark.parametrize("precision", [etm.ETM_PREC_FP64, etm.ETM_PREC_MIXED])
def test_coefficient_refresh_long_chunks(precision):
    prob = W.random_problem(9, 254, 1199, 30, n_steps=8, R=2, n_ports=4, amp=3e10)
    dt = etm.cfl_dt(prob)
    J = prob.sample_J_half(dt, 8)
    plan = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=8, history=False)
    plan.advance(4)
    plan.sync()
    again = etm.Plan(prob, J, dt=dt, precision=precision, n_steps=8, history=False)
    again.restore(plan.checkpoint())
    out = []
    for p in (plan, again):
        p.advance(4)
        p.sync()
        out.append(p.e() + [p.read(etm.ETM_FIELD_THETA)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert np.abs(out[0][3]).max() > 0
