"""The transpose of the ray sums over up to four angles, which takes the
sinogram as it is: the same bits as the general path gives for these angles
and others whose samples are zero, parity, and a sinogram that is not finite
in one angle (as in the general path, corners that this angle does not see
keep the others' values)."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, make_problem
from tests.test_gpu_ray_transpose import _adj, _w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(64, 64), (128, 64), (64, 192), (64, 1024)])
@pytest.mark.parametrize("k0,k", [(0, 1), (2, 2), (1, 3), (3, 4)])
def test_the_same_bits_as_the_general_path(H, W, k0, k):
    theta = np.array([0, 0.25, 0.5, 1.1, -0.7, 2.3, 0.75, 1.0, 0.1, 0.33]) * np.pi
    p = make_problem(H, W, 2, config=68, mag_rel=(1.0,))
    g = p.geom
    p.geom = O.Geometry(H=H, W=W, theta=theta, mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0, kappa=g.kappa)
    p.chunk = 4
    w = _w(p, 7, 5)
    w[k:] = 0
    few = _adj(p, w[:k].copy(), k0, k0 + k)
    assert (few == _adj(p, w, k0, k0 + 7)).all()
    if W <= 192:
        sub = O.Geometry(H=H, W=W, theta=theta[k0:k0 + k], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                         kappa=g.kappa)
        gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w[:k]), sub)
        assert_close(few, gu, "g_u")


@pytest.mark.parametrize("n", [2, 6])               # the short path and the general one
@pytest.mark.parametrize("e", [-40, 40])
def test_an_angle_that_is_not_finite(n, e):
    W = 64
    p = make_problem(64, W, n, config=69, chunk=4, mag_rel=(1.0,), theta=np.array([0.0, 0.25] + [0.0] * (n - 2)) * np.pi)
    w = _w(p, n, 6) * np.float32(2.0 ** e)
    g = p.geom
    keep = [k for k in range(n) if k != 1]
    sub = O.Geometry(H=64, W=W, theta=g.theta[keep], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0, kappa=g.kappa)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w[keep]), sub)
    w[1, 0, 20, 30] = np.nan
    out = _adj(p, w, 0, n)
    y, x = np.meshgrid(np.arange(W), np.arange(W), indexing="ij")
    s = W / 2 + (x + y - W) * np.sqrt(0.5)
    clear = (s < -8) | (s > W + 8)
    assert not np.isfinite(out[:, W // 2, W // 2]).any()
    assert_close(out[:, clear] * 2.0 ** -e, gu[:, clear] * 2.0 ** -e, "g_u in the corners")
