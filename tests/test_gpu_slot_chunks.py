"""The slots of the probe-gradient sums over several chunks: set by the first
chunk, added to by the next, the last chunk smaller than the number of slots
(some of its shares are empty), in every kind of pass that fills them.  Chunks
below 32 angles are taken as they are, so the calls do take several."""

import numpy as np
import pytest

from tests.problems import assert_close, assert_close_scalar, gpu_plan, make_problem, oracle_grad, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "padded", "probe shifts"])
@pytest.mark.parametrize("H,W,angles,chunk", [(64, 64, 35, 31), (64, 128, 35, 17), (128, 64, 9, 4)])
def test_gradient_over_several_chunks(H, W, angles, chunk, kind):
    p = make_problem(H, W, angles, config=67, chunk=chunk, mag_rel=(1.0, 1.25))
    if kind == "padded":
        p.geom.pad = 2
    elif kind == "probe shifts":
        rng = np.random.default_rng(4)
        p.geom.probe_shift = rng.uniform(-3, 3, (angles, 2, 2)).astype(np.float32).astype(np.float64)
    F, gu, gq = oracle_grad(p)
    plan = gpu_plan(p)
    if kind == "padded":
        plan.set_padding(2)
    elif kind == "probe shifts":
        plan.set_probe_shifts(p.geom.probe_shift)
    plan.workspace("cuda:0").fill_(255)
    args = to_gpu(p)
    for _ in range(2):
        plan.timing(True)
        gF, g_u, g_q = plan.holo_grad(*args)
        chunks = plan.kernel_times()["pass_c"][1] / (1 if kind == "plain" else 2)
        plan.timing(False)
        assert chunks == len(_chunks(plan.ray_groups(), chunk)) > 1
        assert_close_scalar(gF.item(), F)
        assert_close(g_u.cpu().numpy(), gu, "g_u")
        assert_close(g_q.cpu().numpy(), gq, "g_q")


def _chunks(groups, most):
    """Whole groups of angles, at most `most` to a chunk."""
    out = [0]
    for _, n in groups:
        if out[-1] + n > most:
            out.append(0)
        out[-1] += n
    return out
