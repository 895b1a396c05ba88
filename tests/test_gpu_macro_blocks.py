"""The macroscopic prediction on velocity grids at the edges of its half-space
sums (one and two 64-column scans, odd counts, n1 != n2) and on meshes with
faces along the axes, against the oracle after the same sweeps.  Both sides
evaluate the same sums in FP64 in another order: 1e-11 of max|.| as in the
acceleration tests; the adjoint's correction uses the same blocks."""
import numpy as np
import pytest

import oracle
from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm  # noqa: E402
from _parity import _rel, check_resid  # noqa: E402


def _square(n):
    """An O-grid whose inner and outer walls are squares: faces along x and y."""
    g = I.ogrid(n, 6, 4.0, 1.1)
    p = g.nodes
    r = np.hypot(p[..., 0], p[..., 1])
    g.nodes = p * (r / np.maximum(np.abs(p[..., 0]), np.abs(p[..., 1])))[..., None]
    return g


@pytest.mark.parametrize("n1,n2", [(16, 16), (17, 24), (64, 16), (65, 18), (128, 16), (16, 70)])
@pytest.mark.parametrize("mesh", ["square", "airfoil"])
def test_prediction(n1, n2, mesh):
    g = _square(16) if mesh == "square" else I.naca_cgrid(4, 8, 6, t=0.12, m=0.02, r_outer=4.0, h1=0.03)
    wl = I.Workload("blocks", g, I.VGridSpec(I.VG_MIDPOINT, n1, n2, 5.0), I.FlowSpec(0.05, 0.6, 1.1), 0)
    s = dvm.Solver.from_workload(wl, equilibrium=dvm.EQ_CONSERVATIVE, accelerate=(3, 12))
    o = oracle.Problem.from_workload(wl, nthreads=8)
    o.set_equilibrium(dvm.EQ_CONSERVATIVE)
    o.set_acceleration(3, 12)
    s.primal_init()
    _, r = s.primal_iterate(7)
    o.primal_init()
    ro = o.primal_iterate(7)
    check_resid(r, ro, "primal")
    assert _rel(s.state_array(dvm.STATE_F), o.f) <= 1e-11
    assert _rel(s.moments(), o.W) <= 1e-11
    s.adjoint_init()
    _, ra = s.adjoint_iterate(7)
    o.adjoint_init()
    rao = o.adjoint_iterate(7)
    check_resid(ra, rao, "adjoint")
    assert _rel(s.state_array(dvm.STATE_PHI), o.phi) <= 1e-11
