"""The Fourier-slice projector's own part of the workspace: at most 384 MB, or
what eight slices need where that is more, however many angles a plan has."""

import numpy as np
import pytest

from paper_2407_20304_amd import holo, synth
from tests.test_fs_shares import shares


@pytest.mark.parametrize("H,W,n", [(64, 64, 20000), (128, 128, 2000), (512, 64, 2000), (64, 256, 3000), (64, 1024, 8)])
def test_bound(H, W, n):
    theta = np.arange(n) * np.pi / n
    p = holo.Plan(H, W, theta, [1.0], synth.M0, synth.FRESNEL0, synth.KAPPA, chunk=4)
    p.set_projector("fourier")
    frame = H * W * 8
    # probe, its gradient's slots (one per angle of the chunk), the reference,
    # psi and X; sinogram; cost slots and the rest
    other = frame * (1 + 4 + 1 + 4 + 4) + H * (W + 64) * 8 * n + (W // 4) * 8 * (n + 1) + (1 << 20)
    eight = 8 * (2 * W) ** 2 * 8 + 8 * n * (W + 1) * 8 + 16384 * int(shares(W, theta, 2 * np.pi / 4096))
    assert p.workspace_bytes <= other + max(384 << 20, eight)
    p.close()
