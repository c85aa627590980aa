"""Chunks of at least 32 angles whose frames are small run several at a time:
one chunk below and at the limit, a join that ends inside the angles, a range
of angles, the two ray-sum buffers, probe shifts.  A join leaves every
per-angle result as it is."""

import numpy as np
import pytest

from tests.problems import assert_close, assert_close_scalar, gpu_plan, make_problem, oracle_grad_many, oracle_threads, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,angles,chunk,kind", [
    (64, 64, 70, 31, "plain"),            # below the limit: three chunks
    (64, 64, 70, 32, "plain"),
    (64, 64, 70, 32, "overlap"),
    (64, 64, 70, 32, "probe shifts"),
    (256, 256, 70, 32, "plain"),          # two chunks fit 128 MB: 64 angles, then 6
    (256, 256, 70, 32, "overlap"),
])
def test_gradient(H, W, angles, chunk, kind):
    p = make_problem(H, W, angles, config=47, chunk=chunk, threads=oracle_threads())
    if kind == "probe shifts":
        rng = np.random.default_rng(5)
        shape = (angles, len(p.geom.mag_rel), 2)
        p.geom.probe_shift = rng.uniform(-3, 3, shape).astype(np.float32).astype(np.float64)
    F, gu, gq = oracle_grad_many(p)
    plan = gpu_plan(p)
    if kind == "overlap":
        plan.set_tile("overlap", 1)
    elif kind == "probe shifts":
        plan.set_probe_shifts(p.geom.probe_shift)
    plan.workspace("cuda:0").fill_(255)
    u, q, amp, ref = to_gpu(p)
    gF, g_u, g_q = plan.holo_grad(u, q, amp, ref)
    assert_close_scalar(gF.item(), F)
    assert_close(g_u.cpu().numpy(), gu, "g_u")
    assert_close(g_q.cpu().numpy(), gq, "g_q")
    # the same kernel (ray sums in 8-bin blocks) on the same groups of angles
    # gives the same fields whatever goes together
    few = gpu_plan(p)
    few.set_chunk(8)
    assert few.chunk == 8 and plan.chunk == chunk
    for pl in (plan, few):
        pl.set_tile("fwd_bins", 8)
        if kind == "probe shifts":
            pl.set_probe_shifts(p.geom.probe_shift)
    assert few.workspace_bytes < plan.workspace_bytes
    v = plan.holo_fwd(u, q).cpu().numpy()
    assert bool((v == few.holo_fwd(u, q).cpu().numpy()).all())
