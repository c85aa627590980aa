"""The spread of the Fourier-slice transpose shares out the tiles that many
lines meet, counted from the plan's own angles: in a scan over a wedge the
tiles along it meet far more lines than in a full one.  Seen through the
workspace, which holds 16 KB (256 points of 8 slices) per share; on the GPU,
parity over a wedge."""

import numpy as np
import pytest

from oracle import holo_oracle as O
from paper_2407_20304_amd import holo, synth
from tests.problems import assert_close, c128, gpu_plan, make_problem

SHARE, REACH = 128, 12 * np.sqrt(2) + 0.05      # lines of a share; from a tile's centre


def shares(W, theta, spare):
    """Shares of all shared tiles if a line meets a tile within REACH (plus
    `spare` radians) of its centre or of an image that samples reach."""
    M = 2 * W
    c = np.arange(0, M, 16) - M / 2 + 7.5
    t = np.sort(np.mod(theta, np.pi))
    t = np.concatenate([t - np.pi, t, t + np.pi])
    most = np.zeros((len(c), len(c)), int)
    for oy in (-M, 0, M):
        for ox in (-M, 0, M):
            x, y = np.meshgrid(c + ox, c + oy)
            rc = np.hypot(x, y)
            dl = np.arcsin(np.minimum(1, REACH / rc)) + spare
            phi = np.mod(np.arctan2(y, x), np.pi)
            n = np.searchsorted(t, phi + dl, "right") - np.searchsorted(t, phi - dl, "left")
            n = np.minimum(np.where(rc <= REACH, len(theta), n), len(theta))
            most = np.maximum(most, np.where(rc <= W + REACH, n, 0))
    parts = -(-most // SHARE)
    return parts[parts > 1].sum()


@pytest.mark.parametrize("n", [450, 2000])
def test_a_wedge_is_shared_by_its_own_lines(n):
    W = 512
    full, wedge = np.arange(n) * np.pi / n, 0.6 + np.arange(n) * 0.2 / n
    need = []
    for theta in (full, wedge):
        p = holo.Plan(64, W, theta, [1.0], synth.M0, synth.FRESNEL0, synth.KAPPA, chunk=4)
        p.set_projector("fourier")
        need.append(p.workspace_bytes)
        p.close()
    more = (need[1] - need[0]) / (256 * 8 * 8)
    spare = 2 * np.pi / 4096                      # at most two bins of the angle table on each side
    lo = shares(W, wedge, 0) - shares(W, full, spare)
    hi = shares(W, wedge, spare) - shares(W, full, 0)
    assert lo > 0 and lo <= more <= hi, (lo, more, hi)


@pytest.mark.gpu
@pytest.mark.parametrize("W,n,width", [(64, 300, 0.2), (128, 140, 0.01), (64, 140, 0.0)])
def test_adjoint_over_a_wedge(W, n, width):
    import torch
    theta = 3.0 + np.arange(n) * (width / n)      # across the end of the half-turn where wide
    p = make_problem(64, W, 2, config=66, mag_rel=(1.0,))
    g = p.geom
    p.geom = O.Geometry(H=64, W=W, theta=theta, mag_rel=g.mag_rel, m0=g.m0, fresnel0=g.fresnel0, kappa=g.kappa,
                        projector="fourier")
    rng = np.random.default_rng(3)
    w = (rng.standard_normal((n, 1, 64, W)) + 1j * rng.standard_normal((n, 1, 64, W))).astype(np.complex64)
    gu, _ = O.adjoint(c128(p.u), c128(p.q), c128(w), p.geom)
    plan = gpu_plan(p)
    plan.set_projector("fourier")
    dev = torch.device("cuda:0")
    plan.workspace(dev).fill_(255)
    g_u, _ = plan.holo_adj(torch.from_numpy(p.u).to(dev), torch.from_numpy(p.q).to(dev), torch.from_numpy(w).to(dev),
                           0, n, want_q=False)
    assert_close(g_u.cpu().numpy(), gu, "g_u")
