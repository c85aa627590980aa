"""The forward's row windows: only the columns that a row's taps read are
staged, and only the rows whose window meets the volume are walked.  Angles
at the axes, next to the 45 degree switch and steep in every quadrant (rows
outside the volume at either end, windows cut by its edge), single angles
and full groups, 8- and 16-bin workgroups."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, gpu_plan, make_problem

pytestmark = pytest.mark.gpu

EDGE = np.array([0.0, 1e-9, np.pi / 4 - 1e-6, np.pi / 4, np.pi / 4 + 1e-6, np.pi / 2, 2.2, 3 * np.pi / 4,
                 3.0, np.pi, -0.8, -2.4])
STEPS = np.arange(9) * 0.004 + 0.77      # full groups around the switch


@pytest.mark.parametrize("W", [64, 384])
@pytest.mark.parametrize("bins", [16, 8])
@pytest.mark.parametrize("theta", [EDGE, STEPS], ids=["edges", "steps"])
def test_fields(W, bins, theta):
    import torch
    p = make_problem(64, W, 2, config=46, mag_rel=(1.0,))
    # every voxel carries weight, the outermost ones too
    rng = np.random.default_rng(9)
    u = (rng.uniform(0, 2e-6, p.u.shape) * (1 + 0.01j)).astype(np.complex64)
    g = p.geom
    p.geom = O.Geometry(H=64, W=W, theta=theta, mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0,
                        kappa=g.kappa)
    v0 = O.forward(c128(u), c128(p.q), p.geom)
    plan = gpu_plan(p)
    plan.set_tile("fwd_bins", bins)
    dev = torch.device("cuda:0")
    plan.workspace(dev).fill_(255)
    v = plan.holo_fwd(torch.from_numpy(u).to(dev), torch.from_numpy(p.q).to(dev))
    assert_close(v.cpu().numpy(), v0, "v")
