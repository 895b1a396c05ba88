"""Macroscopic prediction where the two sides of the O-grid's seam or of the
C-grid's wake cut hold their nodes separately and not to the same digits (a
grid file with rounded numbers): the residual's moments are those of the
sweep, whose faces take each cell's own face vector, so the accelerated
iteration still ends in the plain iteration's solution.

Both run until a sweep changes the moments by less than 1e-12.  The slowest mode (some
thousand sweeps) leaves the state within 1e3 of that, the drag, a wall integral, as near:
bar 1e-8.  The mismatch itself is 1e-3 of the nodes.
"""
import numpy as np
import pytest

from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm  # noqa: E402
from _parity import _rel, _say  # noqa: E402


def grid(kind):
    if kind == "o":
        g = I.ogrid(20, 12, 4.0, 1.2, np.array([0.0, 0.02, 0.01, 0.0]), np.array([0.01, 0.0, 0.02, 0.0]))
        moved = g.nodes[1:, g.ni]                                   # off the wall
    else:
        g = I.naca_cgrid(6, 10, 10, t=0.12, m=0.02, r_outer=5.0, h1=0.05)
        moved = g.nodes[0, g.ni - g.n_wake + 1:]                    # the cut's upper side
    moved[...] = np.round(moved * (1.0 + 1e-3), 3)
    return g


@pytest.mark.parametrize("kind", ["o", "c"])
@pytest.mark.parametrize("batched", [False, True])
def test_mismatched_seam(kind, batched):
    wl = I.Workload("seam", grid(kind), I.VGridSpec(I.VG_MIDPOINT, 12, 12, 5.0), I.FlowSpec(0.1, 0.5, 1.1), 0)
    out = []
    for acc in (None, (5, 20)):
        s = dvm.Solver.from_workload(wl, equilibrium=1, accelerate=acc)
        s.primal_init()
        if batched and acc:
            b = dvm.Batch([s])
            b.run(200)
            b.close()
        it, r = s.primal_iterate(20000, tol=1e-12, check_every=20)
        out.append((s.state_array(dvm.STATE_F), s.objective()[0]))
        _say(f"[seam] {kind} accelerate={acc}: {it} sweeps, r {r:.2e}, J {out[-1][1]:.12e}")
    (f, J), (fa, Ja) = out
    assert _rel(fa, f) <= 1e-8
    assert abs(Ja - J) <= 1e-8 * abs(J)
