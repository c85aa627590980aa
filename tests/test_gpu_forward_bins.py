"""Bins per workgroup of the forward ray sums: an angle's fields are the same
bits in every chunk and range of whole groups, also where small launches take
the 16-bin blocks in halves; a value that the caller sets is the one that
runs."""

import numpy as np
import pytest
import torch

from oracle import holo_oracle as O
from paper_2407_20304_amd import synth
from tests.problems import Problem, assert_close, c128, gpu_plan

pytestmark = pytest.mark.gpu


def _problem(W, angles):
    """Every voxel carries weight; a number of angles over the half-turn, or
    the angles.  (No data: the fields alone are looked at.)"""
    theta = np.arange(angles) * (np.pi / angles) if np.ndim(angles) == 0 else angles
    rng = np.random.default_rng(4)
    u = (rng.uniform(0, 2e-6, (64, W, W)) * (1 + 0.01j)).astype(np.complex64)
    geom = O.Geometry(H=64, W=W, theta=theta, mag_rel=(1.0,), m0=synth.M0, fresnel0=synth.FRESNEL0, kappa=synth.KAPPA)
    return Problem(geom, u, synth.probe(64, W, 3), None, None, 0)


def _fields(plan, p, *k):
    dev = torch.device("cuda:0")
    return plan.holo_fwd(torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev), *k).cpu().numpy()


EDGES = np.array([0.0, 1e-9, np.pi / 4 - 1e-6, np.pi / 4, np.pi / 4 + 1e-6, np.pi / 2, 2.2, 3 * np.pi / 4,
                  3.0, np.pi, -0.8, -2.4])


# 64 px: halves in every launch; 512: in short ones; edges: axes, the walk
# switch, windows outside the volume at either end
@pytest.mark.parametrize("W,n", [(64, 90), (512, 70), (192, EDGES), (1024, EDGES[:7]),
                                 (2048, EDGES[2:5])],
                         ids=["64", "512", "192-edges", "1024-edges", "2048-edges"])
def test_the_same_bits_in_every_chunk_and_range(W, n):
    p = _problem(W, n)
    n = len(p.geom.theta)
    whole = gpu_plan(p)
    whole.set_chunk(n)
    whole.set_tile("fwd_bins", 16)
    v = _fields(whole, p)
    plan = gpu_plan(p)
    assert (_fields(plan, p) == v).all()
    groups = plan.ray_groups()
    k0, k1 = groups[max(0, len(groups) - 4)][0], groups[-1][0]
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
    assert (v["16"] == v["default"]).all()
    # groups and windows of 8 bins round their taps differently
    assert (v["8"] != v["default"]).any()
