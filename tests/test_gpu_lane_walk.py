"""Sweeps at the edges of the lane walk (rows of la lanes, padded tables):
velocity grids narrower than, equal to, just above and several times a lane
row, in both precisions, against the oracle after the same sweeps.

FP64: the iterates agree to rounding (a few sweeps of O(100) operations per
value: 1e-11 of max|.|, integrals 1e-10).  FP32 state: 6e-8 per rounding, ten
or so per value and sweep, adding up over the sweeps: 2e-5 of max|f|.
"""
import numpy as np
import pytest

import oracle
from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm  # noqa: E402
from _parity import _rel, check_resid, check_sens  # noqa: E402

GRIDS = [(2, 2), (7, 64), (15, 17), (16, 5), (33, 10), (48, 12), (63, 6), (66, 9), (96, 10), (127, 3), (128, 4)]


@pytest.mark.parametrize("n1,n2", GRIDS)
@pytest.mark.parametrize("precision", [dvm.FP64, dvm.MIXED])
@pytest.mark.parametrize("order", [1, 2])
def test_walk(n1, n2, precision, order):
    g = I.ogrid(9, 5, 4.0, 1.2, np.array([0.0, 0.02, 0.01, 0.0]), np.array([0.01, 0.0, 0.02, 0.0]))
    wl = I.Workload("walk", g, I.VGridSpec(I.VG_MIDPOINT, n1, n2, 3.0), I.FlowSpec(0.8, 0.4, 1.1), 0)
    s = dvm.Solver.from_workload(wl, precision=precision, order=order, correction_every=4)
    o = oracle.Problem.from_workload(wl, nthreads=8)
    if order == 2:
        o.set_scheme(2, True, 4)
    s.primal_init()
    _, r = s.primal_iterate(6)
    o.primal_init()
    ro = o.primal_iterate(6)
    s.adjoint_init()
    _, ra = s.adjoint_iterate(5)
    o.adjoint_init()
    rao = o.adjoint_iterate(5)
    fp64 = precision == dvm.FP64
    assert _rel(s.state_array(dvm.STATE_F), o.f) <= (1e-11 if fp64 else 2e-5)
    assert _rel(s.moments(), o.W) <= (1e-11 if fp64 else 2e-5)
    J, Jo = s.objective()[0], o.objective()
    assert abs(J - Jo) <= (1e-10 if fp64 else 2e-5) * abs(Jo)
    if fp64:
        check_resid(r, ro, "primal")
        check_resid(ra, rao, "adjoint")
        assert _rel(s.state_array(dvm.STATE_PHI), o.phi) <= 1e-11
        check_sens(s.wall_sensitivity(), o.wall_sensitivity(), 1e-10)
        if order == 1:
            assert _rel(s.mesh_sensitivity(), o.mesh_sensitivity()) <= 1e-10


@pytest.mark.parametrize("n1,n2", [(16, 5), (33, 10), (96, 10)])
@pytest.mark.parametrize("precision", [dvm.FP64, dvm.MIXED])
def test_reloaded_state_continues_bitwise(n1, n2, precision):
    """The moments of a loaded f and of a loaded phi are the sweeps' own."""
    wl = I.Workload("walk", I.ogrid(9, 5, 4.0, 1.2), I.VGridSpec(I.VG_MIDPOINT, n1, n2, 4.0), I.FlowSpec(0.8, 0.6), 0)
    s = dvm.Solver.from_workload(wl, precision=precision)
    s.primal_init()
    s.primal_iterate(4)
    W, f = s.moments(), s.state_save(dvm.STATE_F)
    s.state_load(dvm.STATE_F, f)
    assert np.array_equal(s.moments(), W)
    s.adjoint_init()
    s.adjoint_sweeps(3)
    rows = s.state_save(dvm.STATE_PHI_ROWS)
    s.adjoint_sweeps(2)
    want = s.state_save(dvm.STATE_PHI)
    s.state_load(dvm.STATE_PHI_ROWS, rows)
    s.adjoint_sweeps(2)
    assert np.array_equal(s.state_save(dvm.STATE_PHI), want)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("ni,nj,n", [(64, 64, 32), (128, 64, 32), (128, 128, 32), (200, 129, 33)])
def test_cache_rule_does_not_change_results(ni, nj, n, adjoint):
    """Solves whose rows fit the memory-side cache, nearly fit it (every other
    sweep backwards) and do not, alone and in a batch of four with another
    rule: the bits stay the same."""
    wl = I.circle_case(ni, nj, n, 5.0, 0.8, 0.6)
    one = dvm.Solver.from_workload(wl, want_adjoint=adjoint)
    many = [dvm.Solver.from_workload(wl, want_adjoint=adjoint) for _ in range(4)]
    which = dvm.STATE_PHI if adjoint else dvm.STATE_F
    for s in [one] + many:
        s.primal_init()
        if adjoint:
            s.primal_sweeps(2)
            s.adjoint_init()
    (one.adjoint_sweeps if adjoint else one.primal_sweeps)(3)
    b = dvm.Batch(many)
    b.run(3)
    b.close()
    want = one.state_save(which)
    for s in many:
        assert np.array_equal(s.state_save(which), want)


# (cells, velocities, precision): rows in 4 and in 2 parts for few cells, FP64
# rows from memory in 4 parts, FP32 ones with only the last patches in parts
@pytest.mark.parametrize("ni,nj,n1,n2,precision", [
    (17, 9, 24, 24, dvm.FP64), (30, 21, 17, 20, dvm.MIXED), (45, 33, 24, 24, dvm.FP64), (40, 30, 33, 31, dvm.MIXED),
    (120, 50, 47, 49, dvm.FP64), (130, 63, 64, 66, dvm.MIXED)])
def test_rows_in_parts(ni, nj, n1, n2, precision):
    """Sweeps whose rows several waves share, against the oracle, and bit for
    bit the batch's, where one wave takes all parts."""
    g = I.ogrid(ni, nj, 6.0, 1.05, np.array([0.0, 0.02, 0.01, 0.0]), np.zeros(4))
    wl = I.Workload("parts", g, I.VGridSpec(I.VG_MIDPOINT, n1, n2, 4.0), I.FlowSpec(0.8, 0.4, 1.1), 0)
    s, m = [dvm.Solver.from_workload(wl, precision=precision) for _ in range(2)]
    o = oracle.Problem.from_workload(wl, nthreads=16)
    o.primal_init()
    ro = o.primal_iterate(3)
    for x in (s, m):
        x.primal_init()
    _, r = s.primal_iterate(3)
    b = dvm.Batch([m])
    b.run(3)
    assert abs(b.residuals()[0] - r) <= 1e-12 * r
    b.close()
    assert np.array_equal(s.state_save(dvm.STATE_F), m.state_save(dvm.STATE_F))
    assert np.array_equal(s.moments(), m.moments())
    tol = 1e-11 if precision == dvm.FP64 else 2e-5
    assert _rel(s.moments(), o.W) <= tol
    W = s.moments()
    s.state_load(dvm.STATE_F, s.state_save(dvm.STATE_F))
    assert np.array_equal(s.moments(), W)
    for x in (s, m):
        x.adjoint_init()
    _, ra = s.adjoint_iterate(2)
    b = dvm.Batch([m])
    b.run(2)
    assert abs(b.residuals()[0] - ra) <= 1e-12 * ra
    b.close()
    assert np.array_equal(s.state_save(dvm.STATE_PHI), m.state_save(dvm.STATE_PHI))
    o.adjoint_init()
    o.adjoint_iterate(2)
    if precision == dvm.FP64:
        check_resid(r, ro, "primal")
        assert _rel(s.state_array(dvm.STATE_PHI), o.phi) <= 1e-11
