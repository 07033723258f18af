"""The rule that chooses between the two multi-workgroup CSR kernels, on the host: a grid that the device cannot hold
at once in the two-exchange kernel goes to the one with grid barriers (a device or partition of few CUs)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include "rsk_kernels.hpp"
#include <stdio.h>
int main() {
  using rsk::csr_one_pass;
  int bad = 0;
  auto want = [&](int eta, int G, int resident, bool one) {
    if (csr_one_pass(eta, G, resident) != one) { printf("eta %d G %d resident %d\n", eta, G, resident); ++bad; }
  };
  want(2048, 256, 1280, true);   // a whole MI355X: five workgroups a CU
  want(2048, 256, 160, false);   // 32 CUs
  want(2048, 256, 256, true);
  want(2048, 256, 255, false);
  want(2049, 256, 1280, false);  // a second pass
  want(2049, 257, 1280, false);  // more exchange words than the kernel polls
  want(512, 64, 160, true);
  want(512, 64, 0, true);        // no device: the layout of the whole one
  return bad;
}
"""


@pytest.mark.timeout(300)
def test_csr_route_follows_the_kernels_own_residency(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("ROCm compiler not installed")
    src, exe = tmp_path / "route.cpp", tmp_path / "route"
    src.write_text(PROGRAM)
    cc = shutil.which("g++")
    r = subprocess.run([cc, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                        f"-I{ROOT}/paper_2203_10838_amd/csrc", str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
