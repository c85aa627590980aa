"""The Fourier-slice projector where its work items and slabs can go wrong:
tiles shared between workgroups (more lines than one takes), several slabs
per launch with fewer slices than a slab holds, ranges of unsorted angles."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, gpu_plan, make_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,n,k0,k1,slab,order", [
    (64, 64, 300, 0, 300, 8, "uniform"),
    (64, 64, 150, 20, 149, 4, "scattered"),
    (128, 64, 5, 1, 3, 2, "scattered"),
    (64, 192, 3, 0, 3, 8, "uniform"),
])
def test_forward_and_adjoint(H, W, n, k0, k1, slab, order):
    import torch
    theta = np.arange(n) * (np.pi / n)
    if order == "scattered":
        theta = np.random.default_rng(3).uniform(-2 * np.pi, 2 * np.pi, n)
    p = make_problem(H, W, 2, config=45, mag_rel=(1.0,))
    g = p.geom
    p.geom = O.Geometry(H=H, W=W, theta=theta, mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                        kappa=g.kappa, projector="fourier")
    p.chunk = 64
    rng = np.random.default_rng(6)
    shape = (k1 - k0, 1, H, W)
    w = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    sub = O.Geometry(H=H, W=W, theta=theta[k0:k1], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                     kappa=g.kappa, projector="fourier")
    v0 = O.forward(c128(p.u), c128(p.q), sub)
    gu0, gq0 = O.adjoint(c128(p.u), c128(p.q), c128(w), sub)
    plan = gpu_plan(p)
    plan.set_projector("fourier")
    plan.set_tile("fs_slab", slab)
    dev = torch.device("cuda:0")
    u, q = torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev)
    plan.workspace(dev).fill_(255)
    v = plan.holo_fwd(u, q, k0, k1)
    g_u, g_q = plan.holo_adj(u, q, torch.from_numpy(w).to(dev), k0, k1)
    assert_close(v.cpu().numpy(), v0, "v")
    assert_close(g_u.cpu().numpy(), gu0, "g_u")
    assert_close(g_q.cpu().numpy(), gq0, "g_q")
