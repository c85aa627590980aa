"""Bins per workgroup of the forward ray sums: the plan decides, so an angle's
fields are the same bits in every chunk and range of whole groups, and a
value that the caller sets is the one that runs."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from tests.problems import assert_close, c128, gpu_plan, make_problem

pytestmark = pytest.mark.gpu


def _problem(W, n):
    p = make_problem(64, W, 2, config=63, mag_rel=(1.0,))
    rng = np.random.default_rng(4)
    p.u = (rng.uniform(0, 2e-6, p.u.shape) * (1 + 0.01j)).astype(np.complex64)
    g = p.geom
    p.geom = O.Geometry(H=64, W=W, theta=np.arange(n) * (np.pi / n), mag_rel=g.mag_rel, m0=g.m0,
                        fresnel0=g.fresnel0, kappa=g.kappa)
    return p


def _fields(plan, p, *k):
    import torch
    dev = torch.device("cuda:0")
    return plan.holo_fwd(torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev), *k).cpu().numpy()


@pytest.mark.parametrize("W,n", [(64, 90), (512, 70)])     # 8 bins, 16 bins by default
def test_the_same_bits_in_every_chunk_and_range(W, n):
    p = _problem(W, n)
    plan = gpu_plan(p)
    plan.set_chunk(n)
    v = _fields(plan, p)
    groups = plan.ray_groups()
    k0, k1 = groups[-4][0], groups[-1][0]
    assert (_fields(plan, p, k0, k1) == v[k0:k1]).all()
    for chunk in (4, 17, 31):
        plan.set_chunk(chunk)
        assert (_fields(plan, p) == v).all(), chunk


def test_a_set_value_runs():
    p = _problem(64, 12)
    v0 = O.forward(c128(p.u), c128(p.q), p.geom)
    plan = gpu_plan(p)
    v = {"default": _fields(plan, p)}
    groups = plan.ray_groups()
    plan.set_tile("fwd_bins", 16)
    assert plan.ray_groups() == groups
    v["16"] = _fields(plan, p)
    plan.set_tile("fwd_bins", 8)
    v["8"] = _fields(plan, p)
    for name, x in v.items():
        assert_close(x, v0, name)
    # the default of so small a plan is 8 bins on the groups of 16: the widths
    # round their taps differently
    assert (v["16"] != v["default"]).any()
