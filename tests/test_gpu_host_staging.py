"""Pinned staging of host loads: one buffer of the largest brick for a single
brick, two for more."""
import numpy as np
import pytest

from paper_1205_0282_amd import binding

pytestmark = pytest.mark.gpu


def _mapped():
    """Writable address ranges of this process."""
    with open("/proc/self/maps") as fh:
        lines = [ln.split() for ln in fh]
    return [tuple(int(v, 16) for v in ln[0].split("-")) for ln in lines if ln[1].startswith("rw")]


def _buffers(before, after, size):
    """Buffers of `size` bytes in what was mapped between (neighbours may be one range)."""
    new = []
    for lo, hi in after:
        for a, b in before:
            if lo < b and a < hi:
                if lo < a:
                    new.append(a - lo)
                lo = max(lo, b)
        if lo < hi:
            new.append(hi - lo)
    return sum(n // size for n in new)


@pytest.mark.parametrize("n,brick,buffers", [((401, 403, 397), 512, 1), ((401, 403, 397), 200, 2)])
def test_one_buffer_for_one_brick(n, brick, buffers):
    import torch
    first = np.zeros((8, 8, 8), np.float32)
    vol = np.random.default_rng(2).standard_normal(n[::-1]).astype(np.float32)
    made = []
    for k, v in enumerate((first, vol)):                # (what a process maps once, before)
        bc = binding.BrickCaster(0)
        sizes = bc.plan(v.shape[::-1], (brick,) * 3, storage="f16", max_w=16, max_h=16)
        bc.bind()
        torch.cuda.synchronize()
        before = _mapped()
        bc.load(v)
        added = _buffers(before, _mapped(), sizes[3])
        _, _, mm = bc.bricks()
        assert mm[:, 0].min() == v.min() and mm[:, 1].max() == v.max()
        made.append(bc)
    for bc in made:
        bc.close()
    assert added == buffers
