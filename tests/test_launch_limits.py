"""Host check: the launch that splits the sinogram has fewer than 2^32 threads
(the most that HIP takes in a dimension) for every sinogram a device holds, and
a workgroup for every 256 items of the usual ones."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_20304_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "holo_internal.hpp"
int main() {
  unsigned long long n;
  while (std::scanf("%llu", &n) == 1) std::printf("%u %d\n", holo::split_sino_blocks(n), holo::kThreads);
}
"""


def test_sinogram_split(tmp_path):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(MAIN)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    # items of 32 bytes: the smallest plan, 1024^3 x 1800 angles, 1024^2 x 15500 and 65536 angles, 288 GB
    sizes = [1 * 128 * 16, 1800 * 16 * 1088 * 16, 15500 * 16 * 1088 * 16, 65536 * 16 * 1088 * 16, 288 * 10 ** 9 // 32]
    out = subprocess.run([str(exe)], input="\n".join(map(str, sizes)), capture_output=True, text=True, check=True).stdout
    for n, line in zip(sizes, out.splitlines()):
        blocks, threads = map(int, line.split())
        assert 0 < blocks * threads < 2 ** 32
        assert blocks * threads >= min(n, 2 ** 29)
