"""Calls over fewer angles than the probe-gradient sums have slots: only the
slots of the call's angles are used (one angle: no sum over slots), and those
of earlier, longer calls do not show."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, gpu_plan, make_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "padded", "probe shifts"])
@pytest.mark.parametrize("n", [1, 3, 5])
def test_probe_gradient_of_a_short_range(n, kind):
    import torch
    p = make_problem(64, 64, 40, config=64, chunk=20, mag_rel=(1.0, 1.25))
    g, k0 = p.geom, 7
    rng = np.random.default_rng(n)
    sub = O.Geometry(H=64, W=64, theta=g.theta[k0:k0 + n], mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                     kappa=g.kappa)
    plan = gpu_plan(p)
    if kind == "padded":
        sub.pad = 2
        plan.set_padding(2)
    elif kind == "probe shifts":
        s = rng.uniform(-3, 3, (40, 2, 2)).astype(np.float32)
        sub.probe_shift = s[k0:k0 + n].astype(np.float64)
        plan.set_probe_shifts(s)
    dev = torch.device("cuda:0")
    u, q = torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev)
    w = (rng.standard_normal((40, 2, 64, 64)) + 1j * rng.standard_normal((40, 2, 64, 64))).astype(np.complex64)
    wt = torch.from_numpy(w).to(dev)
    plan.workspace(dev).fill_(255)
    plan.holo_adj(u, q, wt, 0, 40)                 # fills every slot
    plan.timing(True)
    _, g_q = plan.holo_adj(u, q, wt[:n].contiguous(), k0, k0 + n, want_u=False)
    launches = plan.kernel_times()["other"][1]
    plan.timing(False)
    _, gq = O.adjoint(c128(p.u), c128(p.q), c128(w[:n]), sub)
    assert_close(g_q.cpu().numpy(), gq, "g_q")
    # the volume copies, the sum over slots, padded also the sum over planes
    assert launches == 1 + (n > 1) + (kind == "padded")
