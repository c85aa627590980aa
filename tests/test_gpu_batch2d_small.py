"""Batches of 64-px problems on either side of the rule that gives a column
workgroup a whole frame instead of 16 columns (more than 256 workgroups of 16
columns in a pass): gradient, objective and fields, with one plane and several,
alone and next to larger problems."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from paper_2407_20304_amd import synth
from tests.problems import assert_close, assert_close_scalar, c128

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,nd", [((64,) * 16, 4), ((64,) * 17, 4), ((64,) * 65, 1), ((64,) * 3 + (512,) + (64,), 4),
                                      ((64, 128, 64), 2)],
                         ids=["16x4", "17x4", "65x1", "with-512", "with-128"])
def test_batch(sizes, nd):
    import torch
    from paper_2407_20304_amd import holo
    mags = synth.MAG_REL[:nd] if nd > 1 else (1.1,)
    geo = (mags, synth.M0, synth.FRESNEL0)
    rng = np.random.default_rng(5)
    field = lambda *s: (1 + 0.1 * (rng.standard_normal(s) + 1j * rng.standard_normal(s))).astype(np.complex64)
    made = [(field(n, n), field(n, n), np.abs(field(nd, n, n)), np.abs(field(n, n))) for n in sizes]
    dev = torch.device("cuda:0")
    plan = holo.Plan2D(list(sizes), mags, synth.M0, synth.FRESNEL0)
    args = [plan.pack([m[i] for m in made], device=dev) for i in range(4)]
    F, g_psi, g_q = plan.holo2d_grad(*args)
    assert torch.equal(F, plan.holo2d_objective(*args))
    v = plan.unpack(plan.holo2d_fwd(*args[:2]), planes=True)
    g_psi, g_q, F = plan.unpack(g_psi), plan.unpack(g_q), F.cpu().numpy()
    for a in {0, 1, len(sizes) // 2, len(sizes) - 1}:
        psi, q, amp, ref = made[a]
        F0, gp0, gq0 = O.holo2d_gradient(c128(psi), c128(q), amp.astype(np.float64), ref.astype(np.float64), *geo)
        assert_close_scalar(F[a], F0)
        assert_close(g_psi[a].cpu().numpy(), gp0, "g_psi %d" % a)
        assert_close(g_q[a].cpu().numpy(), gq0, "g_q %d" % a)
        assert_close(v[a].cpu().numpy(), O.holo2d_forward(c128(psi), c128(q), *geo), "v %d" % a)
