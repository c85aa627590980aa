"""The transpose of the ray sums on the matrix cores: angle counts that do not
fill its groups of 4 or its set-up windows of 64, first angles past 0, every
quadrant, the smallest slice and tile counts, and the power-of-two scaling of
its split operands (zero and very small sinograms)."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, gpu_plan, make_problem

pytestmark = pytest.mark.gpu


def _adj(p, w, k0, k1):
    import torch
    dev = torch.device("cuda:0")
    plan = gpu_plan(p)
    g_u, _ = plan.holo_adj(torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev),
                           torch.from_numpy(w).to(dev), k0, k1, want_q=False)
    return g_u.cpu().numpy()


def _w(p, n, seed):
    rng = np.random.default_rng(seed)
    g = p.geom
    s = (n, g.n_dist, g.H, g.W)
    return (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)


@pytest.mark.parametrize("H,W,n,k0,k1", [
    (64, 64, 1, 0, 1),
    (64, 64, 9, 3, 8),
    (128, 64, 67, 0, 67),
    (64, 192, 6, 1, 4),
    (64, 64, 140, 5, 134),
])
def test_adjoint_over_angle_ranges(H, W, n, k0, k1):
    # all four quadrants, the axes and the 45 degree walk switch among them
    theta = np.linspace(-0.3, 2 * np.pi, n) if n > 8 else np.array([0, 0.25, 0.5, 1.1, -0.7, 2.3][:n]) * np.pi
    p = make_problem(H, W, n, config=43, chunk=min(n, 32), theta=theta, mag_rel=(1.0,))
    w = _w(p, k1 - k0, 7)
    g = p.geom
    sub = O.Geometry(H=H, W=W, theta=theta[k0:k1], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                     kappa=g.kappa)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w), sub)
    assert_close(_adj(p, w, k0, k1), gu, "g_u")


def test_scaled_sinograms():
    p = make_problem(64, 64, 5, config=44, chunk=4, mag_rel=(1.0, 1.25))
    w = _w(p, 5, 8)
    ref = _adj(p, w, 0, 5)
    assert not _adj(p, 0 * w, 0, 5).any()
    # a power of two goes through every step unchanged
    for e in (-60, 40):
        assert_close(_adj(p, (w * np.float32(2.0 ** e)), 0, 5) * 2.0 ** -e, ref, "scaled by 2^%d" % e, tol=1e-6,
                     max_tol=1e-6)


@pytest.mark.parametrize("H,W,n,nd", [
    (64, 64, 31, 4),       # 8 groups of 4 angles, the last one short: 2 shares
    (64, 64, 77, 8),       # 20 groups: 5 shares
    (128, 128, 37, 4),     # 128 tiles: 2 shares
    (64, 128, 37, 4),      # 64 tiles, 10 groups: 2 shares
])
def test_shared_angles(H, W, n, nd):
    """Volumes of few tiles share their angles out and add the parts up."""
    theta = np.linspace(-0.3, 2 * np.pi, n)
    p = make_problem(H, W, n, config=48, chunk=32, theta=theta, mag_rel=tuple(1 + 0.05 * np.arange(nd)))
    w = _w(p, n, 9)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w), p.geom)
    assert_close(_adj(p, w, 0, n), gu, "g_u")
