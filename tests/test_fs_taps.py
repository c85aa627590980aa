"""Host check of the Fourier-slice projector's tap distances: the header that
the forward and the transpose share, compiled for the host, gives every
distance of a polar sample from a tap in double precision, rounded once."""

import os
import subprocess

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_20304_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "fs_taps.hpp"
int main() {
  int m, M;
  double step;
  while (std::scanf("%d %lf %d", &m, &step, &M) == 3) {
    const holo::FsTap t = holo::fs_tap(m, step, M);
    std::printf("%d", t.i0);
    for (int b = 0; b < holo::kFsWidth; ++b) std::printf(" %.17g", (double)holo::fs_dist(t.r, b));
    std::printf("\n");
  }
}
"""


def test_distances_are_rounded_once(tmp_path):
    src, exe = tmp_path / "taps.cpp", tmp_path / "taps"
    src.write_text(MAIN)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    rng = np.random.default_rng(1)
    m = rng.integers(-512, 513, 4000)
    step = 2 * np.cos(rng.uniform(0, np.pi, 4000))
    text = "\n".join("%d %.17g 2048" % (a, s) for a, s in zip(m, step))
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
    got = np.array([r.split() for r in out.splitlines()], np.float64)
    pos = m * step
    taps = got[:, :1] - 1024 + np.arange(8)
    exact = pos[:, None] - taps
    assert (taps[:, 0] == np.floor(pos) - 3).all()
    assert (np.abs(got[:, 1:] - exact) <= 2.0 ** -24 * np.abs(exact) + 2.0 ** -48).all()
