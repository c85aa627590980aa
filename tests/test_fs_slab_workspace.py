"""The Fourier-slice slab setting changes neither the workspace nor, on the
GPU, the work of a call (slabs always hold 8 slices)."""

import numpy as np
import pytest

from paper_2407_20304_amd import holo, synth


def _plan(H, W, n):
    p = holo.Plan(H, W, np.arange(n) * np.pi / n, synth.MAG_REL, synth.M0, synth.FRESNEL0, synth.KAPPA, chunk=16)
    p.set_projector("fourier")
    return p


@pytest.mark.parametrize("H,W,n", [(64, 64, 90), (192, 128, 33), (64, 1024, 10)])
def test_workspace_is_the_same(H, W, n):
    p = _plan(H, W, n)
    need = p.workspace_bytes
    for slab in (1, 2, 4, 8):
        p.set_tile("fs_slab", slab)
        assert p.get_tile("fs_slab") == slab and p.workspace_bytes == need
    p.close()


@pytest.mark.gpu
def test_time_does_not_grow_below_eight():
    """One slice at a time in records of eight would be eight times the work:
    a factor of two apart tells that from the spread of single runs."""
    import torch
    p = _plan(128, 128, 200)
    u = synth.ellipsoid_volume(128, 128, 1, device="cuda:0")
    q = torch.from_numpy(synth.probe(128, 128, 2)).to("cuda:0")
    w = torch.randn(200, 4, 128, 128, dtype=torch.complex64, device="cuda:0")
    ms = {}
    for slab in (8, 1):
        p.set_tile("fs_slab", slab)
        best = 1e30
        for _ in range(5):
            p.timing(True)
            p.holo_adj(u, q, w, 0, 200)
            t = p.kernel_times()
            best = min(best, t["radon_fwd"][0] + t["radon_adj"][0])
            p.timing(False)
        ms[slab] = best
    print("  ms at 8 and 1 slices:", ms[8], ms[1], flush=True)
    assert ms[1] < 2 * ms[8]
