"""Mesh motion and its transpose for wall sizes at the edges of a block of
eight rows of the triangular solves, against a dense solve in numpy.  The
interpolation matrices here have condition numbers below 1e5, so 1e-10 of the
largest value leaves rounding a factor of ten."""
import numpy as np
import pytest

from paper_2501_00923_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_00923_amd import dvm, shape  # noqa: E402


@pytest.mark.parametrize("nw", [4, 7, 8, 9, 16, 23, 41])
def test_motion_and_chain_match_a_dense_solve(nw):
    g = I.ogrid(nw, 5, 4.0, 1.2, np.array([0.0, 0.02, 0.01, 0.0]), np.zeros(4))
    R = 2.0
    d = shape.Deformer(dvm.Mesh.from_grid(g), R)
    x0, rng = g.nodes, np.random.default_rng(nw)
    c = x0[0, :nw]
    phi = lambda r: np.where(r < 1.0, (1.0 - r) ** 2, 0.0)  # noqa: E731
    M = phi(np.linalg.norm(c[:, None] - c[None], axis=2) / R)
    assert np.linalg.cond(M) < 1e5
    P = phi(np.linalg.norm(x0[..., None, :] - c, axis=3) / R)      # [nj + 1, ni + 1, nw]
    new = c + 0.01 * rng.normal(size=c.shape)
    want = x0 + P @ np.linalg.solve(M, new - c)
    want[0, :nw], want[0, nw] = new, new[0]
    got = d.apply(new)
    assert np.abs(got - want).max() <= 1e-10 * np.abs(want).max()
    s = rng.normal(size=x0.shape)
    h = np.einsum("jiw,jix->wx", P[1:], s[1:])
    back = np.linalg.solve(M, h) + s[0, :nw]
    back[0] += s[0, nw]
    assert np.abs(d.chain(s) - back).max() <= 1e-10 * np.abs(back).max()
