"""Pass C shares a chunk's angles among workgroups, each with its own slot of
the probe-gradient sums: chunks that do not divide into the shares (a last
chunk smaller than their number leaves some empty), a chunk of one angle,
every kind of pass that adds into the slots."""

import numpy as np
import pytest

from tests.problems import assert_close, assert_close_scalar, gpu_plan, make_problem, oracle_grad, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,angles,chunk,mags,kind", [
    (64, 64, 67, 64, (1.0, 1.08, 1.25, 1.5), "plain"),
    (64, 128, 9, 8, (1.0, 1.25), "plain"),
    (128, 64, 5, 4, (1.0,), "probe shifts"),
    (64, 64, 35, 33, (1.0, 1.5), "probe shifts"),
    (64, 64, 35, 33, (1.0, 1.5), "padded"),
])
def test_probe_gradient_over_uneven_shares(H, W, angles, chunk, mags, kind):
    p = make_problem(H, W, angles, config=41, chunk=chunk, mag_rel=mags)
    if kind == "padded":
        p.geom.pad = 2
    elif kind == "probe shifts":
        rng = np.random.default_rng(4)
        p.geom.probe_shift = rng.uniform(-3, 3, (angles, len(mags), 2)).astype(np.float32).astype(np.float64)
    F, gu, gq = oracle_grad(p)
    plan = gpu_plan(p)
    if kind == "padded":
        plan.set_padding(2)
    elif kind == "probe shifts":
        plan.set_probe_shifts(p.geom.probe_shift)
    # the slots of the workspace are set, not added to: any contents will do
    plan.workspace("cuda:0").fill_(255)
    for _ in range(2):
        gF, g_u, g_q = plan.holo_grad(*to_gpu(p))
        assert_close_scalar(gF.item(), F)
        assert_close(g_u.cpu().numpy(), gu, "g_u")
        assert_close(g_q.cpu().numpy(), gq, "g_q")
