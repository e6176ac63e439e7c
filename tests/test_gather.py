"""The threads that gather a host source's bricks (bc_gather.h), on the CPU:
every brick whole in its buffer when it is taken, with two buffers and with
one, and with as many threads as there are."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1205_0282_amd", "csrc")

MAIN = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "bc_gather.h"

int main(int argc, char** argv) {
  if (argc == 2) {
    printf("%d\n", gather_threads(atoll(argv[1])));
    return 0;
  }
  const int n = atoi(argv[1]), n_buffers = atoi(argv[2]), threads = atoi(argv[3]), stride = atoi(argv[4]);
  const int nx = 23, ny = 17, nz = 3 * n;   // bricks of nx - b % 3, ny, 3 voxels, 4 bytes each
  std::vector<uint32_t> src((size_t)nx * stride * (ny + 1) * nz);
  for (size_t i = 0; i < src.size(); ++i) src[i] = (uint32_t)(i * 2654435761u);
  std::vector<Gather::Brick> bricks;
  for (int b = 0; b < n; ++b) {
    Gather::Brick g;
    g.elem = 4 * stride;
    g.row = g.elem * nx;
    g.plane = g.row * (ny + 1);
    g.src = reinterpret_cast<const char*>(src.data()) + 3 * b * g.plane;
    g.rx = nx - b % 3;
    g.ry = ny;
    g.rz = 3;
    g.bytes = 4;
    bricks.push_back(g);
  }
  std::vector<std::vector<uint32_t>> store(n_buffers, std::vector<uint32_t>(nx * ny * 3));
  std::vector<void*> buffers;
  for (auto& s : store) buffers.push_back(s.data());
  long wrong = 0;
  {
    Gather gather(bricks, buffers.data(), n_buffers, threads);
    gather.release(std::min(n, n_buffers));
    for (int b = 0; b < n; ++b) {
      gather.wait(b);
      const uint32_t* got = store[b % n_buffers].data();
      const int rx = nx - b % 3;
      for (int z = 0; z < 3; ++z)
        for (int y = 0; y < ny; ++y)
          for (int x = 0; x < rx; ++x)
            wrong += got[(z * ny + y) * rx + x] != src[((size_t)(3 * b + z) * (ny + 1) + y) * nx * stride + (size_t)x * stride];
      std::fill(store[b % n_buffers].begin(), store[b % n_buffers].end(), 0u);
      if (b + n_buffers < n) gather.release(b + n_buffers + 1);
      if (argc > 5 && b == n / 2) break;   // (given up half-way: the destructor ends the threads)
    }
  }
  printf("%ld\n", wrong);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "g++ is needed"
    d = tmp_path_factory.mktemp("gather")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "gather")
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread", "-I", CSRC, str(d / "main.cpp"), "-o", exe],
                   check=True, timeout=120)
    return exe


@pytest.mark.parametrize("n,buffers", [(1, 1), (2, 2), (9, 1), (9, 2), (10, 2)])
@pytest.mark.parametrize("threads", [0, 1, 8])
@pytest.mark.parametrize("stride", [1, 3])
def test_bricks_are_whole(program, n, buffers, threads, stride):
    for more in ([], ["half"]):
        r = subprocess.run([program] + [str(v) for v in (n, buffers, threads, stride)] + more, capture_output=True,
                           text=True, timeout=60)
        assert r.returncode == 0 and r.stdout.strip() == "0", r.stderr


def test_threads_follow_the_cores_the_process_may_use(program):
    def threads(size, cores=None):
        set_cores = None if cores is None else (lambda: os.sched_setaffinity(0, cores))
        return int(subprocess.run([program, str(size)], capture_output=True, text=True, timeout=60, check=True,
                                  preexec_fn=set_cores).stdout)
    mine = sorted(os.sched_getaffinity(0))
    assert threads(1 << 20) == 0
    for n in {1, min(3, len(mine)), len(mine)}:
        assert threads(1 << 30, set(mine[:n])) == min(8, n)
        assert threads(2 << 20, set(mine[:n])) == min(2, n)
