"""The transpose of the ray sums on sinograms of wide range: samples far below
their slice's largest keep their own precision, and an angle that is not
finite leaves the voxels it does not see as they are."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from paper_2407_20304_amd import synth
from tests.problems import assert_close, c128, gpu_plan, make_problem
from tests.test_gpu_ray_transpose import _adj, _w

pytestmark = pytest.mark.gpu


def test_samples_far_below_the_slice_maximum():
    """An absorbing cylinder: |psi| = 2^-30 on the rays through its axis, 1
    beside it.  The voxels at the axis only meet samples of h that small.  The
    exponent 30 ln 2 is a ray sum of some 50 single-precision additions
    (2^-24 each), which psi and h take up as their relative error."""
    H = W = 64
    p = make_problem(H, W, 12, config=61, chunk=8, mag_rel=(1.0,))
    c = W / 2
    y, x = np.meshgrid(np.arange(W) - c, np.arange(W) - c, indexing="ij")
    r = np.hypot(x, y)
    beta = 30 * np.log(2) / (synth.KAPPA * 40)
    p.u = np.tile(np.where(r < 20, 1e-7 + 1j * beta, 0), (H, 1, 1)).astype(np.complex64)
    w = _w(p, 12, 5)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w), p.geom)
    out = _adj(p, w, 0, 12)
    near = r < 4
    assert np.abs(gu[:, near]).max() < 2.0 ** -24 * np.abs(gu).max()
    tol = 30 * np.log(2) * 50 * 2.0 ** -24
    assert_close(out, gu, "g_u")
    assert_close(out[:, near], gu[:, near], "g_u at the axis", tol=tol, max_tol=tol)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("e", [-40, 0, 40])
def test_an_angle_that_is_not_finite(bad, e):
    """A bad sample of w makes the whole frame of its angle (45 degrees) not
    finite.  The corners along the diagonal project more than 8 bins off the
    detector at that angle: they take the other angle's values, whatever
    their size."""
    H = W = 64
    p = make_problem(H, W, 2, config=62, chunk=2, mag_rel=(1.0,), theta=np.array([0.0, np.pi / 4]))
    w = _w(p, 2, 6) * np.float32(2.0 ** e)
    g = p.geom
    one = O.Geometry(H=H, W=W, theta=g.theta[:1], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                     kappa=g.kappa)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w[:1]), one)
    w[1, 0, 20, 30] = bad
    out = _adj(p, w, 0, 2)
    y, x = np.meshgrid(np.arange(W), np.arange(W), indexing="ij")
    s = W / 2 + (x + y - W) * np.sqrt(0.5)
    clear = (s < -8) | (s > W + 8)
    assert clear.sum() > 20
    assert not np.isfinite(out[:, W // 2, W // 2]).any()
    assert_close(out[:, clear] * 2.0 ** -e, gu[:, clear] * 2.0 ** -e, "g_u in the corners")
