"""The workspace never shrinks as the chunk grows (a caller who sizes it for
the largest chunk of a set can run them all), also where small frames are
taken several chunks at a time."""

import numpy as np
import pytest

from paper_2407_20304_amd import holo, synth


@pytest.mark.parametrize("projector", ["joseph", "fourier"])
@pytest.mark.parametrize("H,W,n", [(64, 64, 400), (192, 192, 300), (256, 256, 360), (192, 384, 300), (64, 1024, 90)])
def test_monotone(H, W, n, projector):
    plan = holo.Plan(H, W, np.arange(n) * np.pi / n, synth.MAG_REL, synth.M0, synth.FRESNEL0, synth.KAPPA)
    plan.set_projector(projector)
    need = []
    for c in (4, 8, 16, 31, 32, 33, 48, 64, 96, 128, 200):
        plan.set_chunk(c)
        need.append(plan.workspace_bytes)
    assert need == sorted(need)
    plan.close()
