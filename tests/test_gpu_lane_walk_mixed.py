"""The FP32 adjoint and its sensitivities on the lane walk (odd and even
rows, padded columns, rows in parts) against the oracle, at the bars of the
other mixed-precision tests: phi 5e-5 of its maximum, wall and exact mesh
sensitivity 1e-3."""
import numpy as np
import pytest

import oracle
from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm  # noqa: E402
from _parity import _rel, _say, check_sens  # noqa: E402


def compare(wl, order, n_primal, n_adjoint):
    s = dvm.Solver.from_workload(wl, precision=dvm.MIXED, order=order, correction_every=4)
    o = oracle.Problem.from_workload(wl, nthreads=16)
    if order == 2:
        o.set_scheme(2, True, 4)
    for x in (s, o):
        x.primal_init()
        x.primal_iterate(n_primal)
        x.adjoint_init()
        x.adjoint_iterate(n_adjoint)
    ep, em = _rel(s.state_array(dvm.STATE_PHI), o.phi), _rel(s.mesh_sensitivity(), o.mesh_sensitivity())
    _say(f"[mixed walk] {wl.vgrid.n1}x{wl.vgrid.n2} order {order}: phi {ep:.2e} mesh sens {em:.2e}")
    assert ep <= 5e-5
    check_sens(s.wall_sensitivity(), o.wall_sensitivity(), 1e-3)
    assert em <= 1e-3


@pytest.mark.parametrize("n1,n2", [(2, 2), (7, 64), (15, 17), (33, 10), (48, 12), (63, 6), (66, 9), (127, 3), (128, 4)])
@pytest.mark.parametrize("order", [1, 2])
def test_walk(n1, n2, order):
    g = I.ogrid(9, 5, 4.0, 1.2, np.array([0.0, 0.02, 0.01, 0.0]), np.array([0.01, 0.0, 0.02, 0.0]))
    compare(I.Workload("walk", g, I.VGridSpec(I.VG_MIDPOINT, n1, n2, 3.0), I.FlowSpec(0.8, 0.4, 1.1), 0), order, 6, 5)


@pytest.mark.parametrize("ni,nj,n1,n2", [(17, 9, 24, 24), (30, 21, 17, 20), (40, 30, 33, 31)])
def test_rows_in_parts(ni, nj, n1, n2):
    g = I.ogrid(ni, nj, 6.0, 1.05, np.array([0.0, 0.02, 0.01, 0.0]), np.zeros(4))
    compare(I.Workload("parts", g, I.VGridSpec(I.VG_MIDPOINT, n1, n2, 4.0), I.FlowSpec(0.8, 0.4, 1.1), 0), 1, 3, 3)


def test_last_patches_in_parts():
    """FP32 rows from memory, only the last patches of an XCD in parts (the oracle's mesh
    sensitivity takes too long here)."""
    g = I.ogrid(130, 63, 6.0, 1.05, np.array([0.0, 0.02, 0.01, 0.0]), np.zeros(4))
    wl = I.Workload("tail", g, I.VGridSpec(I.VG_MIDPOINT, 64, 66, 4.0), I.FlowSpec(0.8, 0.4, 1.1), 0)
    s, o = dvm.Solver.from_workload(wl, precision=dvm.MIXED), oracle.Problem.from_workload(wl, nthreads=16)
    for x in (s, o):
        x.primal_init()
        x.primal_iterate(3)
        x.adjoint_init()
        x.adjoint_iterate(2)
    assert _rel(s.state_array(dvm.STATE_PHI), o.phi) <= 5e-5
