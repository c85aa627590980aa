"""Host check of the halves that small launches of the forward ray sums take a
16-bin block in (no GPU needed).  A half stages the columns floor(mn) - 1 ..
floor(mx) + 2 of a row for its own 8 bins, at most 26 of them, and forms its
tap positions from the lowest column of the whole block's window.  For every
group that plans form, block, half and row this recomputes both windows and
every tap with the kernel's roundings, and checks that the windows fit and that
a tap and its right neighbour are staged."""

import math

import numpy as np
import pytest

from paper_2407_20304_amd import holo, synth
from tests.test_ray_groups import angle_constants

HALF_SEG, PAD = 26, 32


def check(theta, W):
    plan = holo.Plan(64, W, theta, synth.MAG_REL, synth.M0, synth.FRESNEL0, synth.KAPPA)
    groups = plan.ray_groups()
    plan.close()
    A, B, D = angle_constants(np.asarray(theta, np.float64), W)
    y = np.arange(W, dtype=np.float64)[None, None, :]
    checked = 0
    for first, n in groups:
        Aa, Ba, Da = (x[first:first + n][:, None, None] for x in (A, B, D))
        pos = lambda bins: (Aa + y * Da) + bins * Ba
        s16 = np.arange(0, W, 16, dtype=np.float64)[None, :, None]
        lo16 = np.floor(np.minimum(pos(s16), pos(s16 + 15)).min(axis=0)) - 1
        for half in (0, 8):
            sb = s16 + half
            f = np.minimum(pos(sb), pos(sb + 7)).min(axis=0)
            g = np.maximum(pos(sb), pos(sb + 7)).max(axis=0)
            lo, hi = np.floor(f) - 1, np.floor(g) + 2
            kept = (lo >= -PAD) & (lo <= W + PAD - HALF_SEG)       # windows that are not moved
            dx = lo - lo16
            assert ((dx >= 0) & (dx <= 12))[kept].all()
            assert (hi - lo + 1 <= HALF_SEG)[kept].all()
            # a moved window lies in the padding and misses the volume
            assert ((hi < 0) | (lo >= W))[~kept].all()
            for bin_ in range(8):
                s = half + bin_
                base = Aa + (s16 + (s & ~3)) * Ba
                rel = (base + y * Da - lo16).astype(np.float32)
                q = (rel + np.float32(s & 3) * Ba.astype(np.float32)).astype(np.float64)
                col = np.floor(q) - dx
                ok = (col >= 0) & (col + 1 <= hi - lo)
                assert (ok | ~kept[None]).all(), (first, n, s)
            checked += int(kept.sum()) * n
    return checked


@pytest.mark.parametrize("name", ["vol64_a90", "vol256_a360"])
def test_the_workloads(name):
    wl = synth.WORKLOADS[name]
    assert check(wl.theta, wl.W) > 0


@pytest.mark.parametrize("W", [64, 384, 2048])
def test_walk_switches_and_unsorted_angles(W):
    deg = np.array([0.0, 0.1, 44.8, 45.0, 45.2, 90.0, 90.1, 135.0, 179.9, -46.0, 226.0, 314.9])
    assert check(np.deg2rad(deg), W) > 0
    rng = np.random.default_rng(8)
    assert check(rng.uniform(-math.pi, 2 * math.pi, 12), W) > 0
    assert check(0.77 + 0.004 * np.arange(16), W) > 0
