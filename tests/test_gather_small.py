"""Bricks too small to be worth handing over are gathered by the thread that
loads them (bc_gather.h), however large the source is; on the CPU."""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1205_0282_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "bc_gather.h"

int main() {
  const int64_t big = int64_t(1) << 30;
  // 18^3, 26^3 and 34^3 voxels of 4 bytes, and the limit from both sides
  for (int64_t brick : {int64_t(18 * 18 * 18 * 4), int64_t(26 * 26 * 26 * 4), int64_t(98303), int64_t(98304), int64_t(34 * 34 * 34 * 4)})
    printf("%d ", gather_threads(big, brick) == gather_threads(big) ? 1 : gather_threads(big, brick) == 0 ? 0 : -1);
  printf("%d\n", gather_threads(1 << 20, big));
}
"""


def test_small_bricks_take_no_threads(tmp_path):
    gxx = shutil.which("g++")
    assert gxx, "g++ is needed"
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "small")
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", exe], check=True, timeout=120)
    assert subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout.split() == list("000110")
