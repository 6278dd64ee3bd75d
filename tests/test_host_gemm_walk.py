"""Walk of the persistent GEMM workgroups over the output tiles (csrc/ntp_gemm_addr.h): whatever the number of tiles, the rotated order visits every
tile once and leaves every block on its XCD (no GPU: the header is compiled for the host)."""
import os
import subprocess

from tests.test_host_models import CSRC

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "ntp_gemm_addr.h"
int main() {
  for (int n = 1; n <= 3000; ++n) {
    std::vector<int> seen(n, 0);
    for (int v = 0; v < n; ++v) {
      const int r = ntp_gemm::rotate_walk(v, n);
      if (r < 0 || r >= n || (r & 7) != (v & 7) || seen[r]++) { printf("FAIL %d blocks: %d -> %d\n", n, v, r); return 1; }
      if (n <= 256 && r != v) { printf("FAIL %d blocks: one round is not rotated\n", n); return 1; }
    }
  }
  return 0;
}
"""


def test_rotated_walk_is_a_permutation_that_keeps_the_xcd(tmp_path):
    src, exe = tmp_path / "walk.cpp", str(tmp_path / "walk")
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
