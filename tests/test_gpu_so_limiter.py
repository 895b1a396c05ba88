"""The limiter of the second-order scheme in mixed precision takes the room D
to the neighbourhood's extremes in FP64 from the stored values: the drag of a
loaded state, whose sums are FP64, against the same expressions in numpy
(FP32 where the state's precision rules, FP64 where the limiter does).

Both sides add the same rounded terms, so they differ by FP64 rounding: sums of
1e4 terms, 1e-13 of the terms' absolute sum.  (A rounding of D to FP32 moves
the limiter's FP32 value by a unit in the last place now and then.)
"""
import numpy as np
import pytest

from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm  # noqa: E402
from _parity import _say  # noqa: E402


def centroid_offset(g, c):
    """Face midpoints of wall cell c (row j = 0) minus its centroid."""
    q = [g.nodes[0, c], g.nodes[0, c + 1], g.nodes[1, c + 1], g.nodes[1, c]]
    r = [p - q[0] for p in q]
    a = [r[1][0] * r[2][1] - r[1][1] * r[2][0], r[2][0] * r[3][1] - r[2][1] * r[3][0]]
    cen = q[0] + (a[0] * (r[1] + r[2]) + a[1] * (r[2] + r[3])) / (3.0 * (a[0] + a[1]))
    return [0.5 * (q[e] + q[(e + 1) % 4]) - cen for e in range(4)]


def wall_increment(fc, fn, S, vol, rf, rounded_room=False):
    """FP32 reconstructed wall value minus the cell value, all velocities of
    a cell: fc [nv], fn [4][nv] (fc behind a boundary face), S, rf [4][2]."""
    t = np.float32
    S, rt, iv = S.astype(t), [r.astype(t) for r in rf], t(1.0 / vol)
    gx, gy = np.zeros_like(fc), np.zeros_like(fc)
    for q in range(4):
        b = t(0.5) * (fc + fn[q])
        gx = gx + b * S[q, 0]
        gy = gy + b * S[q, 1]
    gx, gy = gx * iv, gy * iv
    d = np.float64
    hi, lo = np.maximum(fc, fn.max(axis=0)), np.minimum(fc, fn.min(axis=0))
    hi, lo = ((hi - fc).astype(d), (lo - fc).astype(d)) if rounded_room else (hi.astype(d) - fc, lo.astype(d) - fc)
    e2 = (1e-3 * fc.astype(d)) ** 2
    p = np.ones(fc.shape)
    for q in range(4):
        inc = gx.astype(d) * d(rt[q][0]) + gy.astype(d) * d(rt[q][1])
        D = np.where(inc > 0, hi, lo)
        n, m = D * D + e2 + 2.0 * inc * D, D * D + 2.0 * inc * inc + inc * D + e2
        p = np.minimum(p, np.where(m > 0, n / np.where(m > 0, m, 1.0), 1.0))
    p = p.astype(t)
    return ((p * gx) * rt[0][0] + (p * gy) * rt[0][1]).astype(d)


def drag(wl, mesh, v, w, f, **kw):
    """J of the loaded f (FP32 [nc][nv], first component) and the sum of its terms' magnitudes."""
    g, m = wl.grid, mesh.export()
    thw = 0.5 * wl.flow.Tw
    gM = np.exp(-(v ** 2).sum(axis=1) / (2.0 * thw)) / (2.0 * np.pi * thw)
    J = size = 0.0
    for l in range(mesh.nw):
        c = int(m["wall_cell"][l])
        nb, S, A, n = m["nbr"][c], m["S"][c], m["wall_A"][l], m["wall_n"][l]
        fn = np.stack([f[k] if k >= 0 else f[c] for k in nb])
        inc = wall_increment(f[c], fn, S, m["vol"][c], centroid_offset(g, c), **kw)
        vn, s0 = v @ n, v @ S[0]
        out = vn > 0
        D = -(w * vn * gM)[~out].sum()
        H = (w * v[:, 0] * vn * gM.astype(np.float32))[~out] / D
        F = (w * s0 * f[c])[s0 > 0] / A
        dF = (w * vn * inc)[out]
        jp = (w * v[:, 0] * vn * (f[c] + inc))[out]
        J += A * (jp.sum() + (F.sum() + dF.sum()) * H.sum())
        size += A * (np.abs(jp).sum() + np.abs(H).sum() * (np.abs(F).sum() + np.abs(dF).sum()))
    return J, size


def state(wl, mesh, v):
    rng = np.random.default_rng(5)
    g = np.exp(-(v ** 2).sum(axis=1)) / np.pi
    return (g * np.exp(rng.uniform(-1.0, 1.0, (mesh.nc, 1)) + 0.4 * rng.standard_normal((mesh.nc, len(v))))).astype(np.float32)


def workload():
    g = I.ogrid(30, 4, 3.0, 1.2, np.array([0.0, 0.02, 0.01, 0.0]), np.array([0.01, 0.0, 0.02, 0.0]))
    return I.Workload("limiter", g, I.VGridSpec(I.VG_MIDPOINT, 18, 18, 3.0), I.FlowSpec(0.8, 0.4, 1.1), 0)


def test_mixed_limiter_room():
    wl = workload()
    mesh, vg = dvm.Mesh.from_grid(wl.grid), dvm.VGrid.from_spec(wl.vgrid)
    v, w = vg.export()
    f = state(wl, mesh, v)
    s = dvm.Solver(mesh, vg, wl.flow.Kn, wl.flow.Ma, wl.flow.Tw, precision=dvm.MIXED, order=2)
    s.state_load_array(dvm.STATE_F, np.stack([f, f], axis=2))
    J, (Jn, size) = s.objective()[0], drag(wl, mesh, v, w, f)
    _say(f"[limiter] J {J:.16e} numpy {Jn:.16e} difference {abs(J - Jn):.2e} of {size:.3e}")
    assert abs(J - Jn) <= 1e-13 * size
