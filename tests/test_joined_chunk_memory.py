"""What joining small chunks may cost: everything held per angle stays within
160 MB (or the caller's chunk), beside the slots of the probe-gradient sums;
on the GPU, candidates that take the same angles together are timed once."""

import numpy as np
import pytest

from paper_2407_20304_amd import holo, synth
from tests.problems import gpu_plan, make_problem, to_gpu


@pytest.mark.parametrize("H,W,n,nd", [(64, 64, 5000, 1), (64, 64, 720, 4), (128, 128, 720, 4), (192, 256, 500, 2)])
@pytest.mark.parametrize("shifts", [False, True])
@pytest.mark.parametrize("overlap", [0, 1])
def test_growth_is_bounded(H, W, n, nd, shifts, overlap):
    p = holo.Plan(H, W, np.arange(n) * np.pi / n, np.linspace(1, 1.5, nd), synth.M0, synth.FRESNEL0, synth.KAPPA)
    p.set_tile("overlap", overlap)
    if shifts:
        p.set_probe_shifts(np.ones((n, nd, 2), np.float32))
    frame = H * W * 8
    per_angle = frame * (nd + 1 + overlap + (nd if shifts else 0))
    p.set_chunk(4)
    # everything but the four angles and their (at least one) slot of frames
    fixed = p.workspace_bytes - 4 * per_angle
    for chunk in (32, 64, 100):
        p.set_chunk(chunk)
        assert p.chunk == chunk
        assert p.workspace_bytes <= fixed + max(160 << 20, chunk * per_angle) + 31 * nd * frame
    p.close()


@pytest.mark.gpu
def test_candidates_that_run_alike_share_a_time():
    p = make_problem(64, 64, 150, config=65, chunk=64, mag_rel=(1.0, 1.25))
    plan = gpu_plan(p)
    best, ms = plan.autotune(*to_gpu(p), candidates=(16, 32, 64, 128))
    assert ms[32] == ms[64] == ms[128] != ms[16]
    assert best == (32 if ms[32] < ms[16] else 16) == plan.chunk
    plan.set_projector("fourier")
    _, ms = plan.autotune_tile("fs_slab", *to_gpu(p), [2, 4, 8])
    assert ms[2] == ms[4] == ms[8]
