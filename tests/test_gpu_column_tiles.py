"""Column and row passes that hold whole tiles in flight: every padded length
(even and uneven plans, one and several wavefronts to a column, the residual
on the kept centre alone) and the probe-gradient columns up to the longest."""

import pytest

from tests.problems import assert_close, assert_close_scalar, gpu_plan, make_problem, oracle_grad, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,pad", [
    (64, 64, 2), (128, 192, 2), (192, 64, 2), (256, 128, 2), (384, 64, 2), (512, 64, 2), (1024, 64, 2),
    (64, 384, 2), (64, 512, 2),
    (192, 64, 1), (384, 64, 1), (1024, 64, 1), (2048, 64, 1), (64, 512, 1),
])
def test_gradient_and_objective(H, W, pad):
    p = make_problem(H, W, 2, config=51, mag_rel=(1.0, 1.25))
    p.geom.pad = pad
    F, gu, gq = oracle_grad(p)
    plan = gpu_plan(p)
    plan.set_padding(pad)
    plan.workspace("cuda:0").fill_(255)
    u, q, amp, ref = to_gpu(p)
    gF, g_u, g_q = plan.holo_grad(u, q, amp, ref)
    assert_close_scalar(gF.item(), F)
    assert_close(g_u.cpu().numpy(), gu, "g_u")
    assert_close(g_q.cpu().numpy(), gq, "g_q")
    assert_close_scalar(plan.holo_objective(u, q, amp, ref).item(), F)
