"""FP8 bricks narrow along x, on both sides of the width from which whole rows
are staged: every stored byte, with sources of both types and with strides."""
import numpy as np
import pytest

from oracle import encoders
from oracle import raycast as rc
from paper_1205_0282_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("src", ["f32", "f16"])
@pytest.mark.parametrize("dims,brick,stride", [
    ((3, 70, 90), (1, 64, 80), 1),       # one micro-block, several workgroups to a brick
    ((5, 9, 6), (2, 3, 5), 2),           # rows of exactly one micro-block
    ((16, 11, 7), (3, 11, 7), 1),        # two, the second with one voxel of its own
    ((76, 10, 9), (38, 5, 9), 1),        # ten micro-blocks
    ((78, 10, 9), (39, 5, 9), 3),        # eleven, rows staged
    ((43, 6, 70), (39, 6, 70), 1),       # the widest brick decides: narrow ones with it
])
def test_stored_bytes_of_narrow_bricks(src, dims, brick, stride):
    import torch
    dt = np.dtype(np.float32 if src == "f32" else np.float16)
    vol = np.random.default_rng(31).standard_normal(dims[::-1]).astype(dt)
    wide = torch.full((dims[2], dims[1] + 1, stride * dims[0]), 6e4, device="cuda",
                      dtype=torch.float32 if src == "f32" else torch.float16)
    wide[:, :dims[1], ::stride] = torch.from_numpy(vol).cuda()
    bc = binding.BrickCaster(0)
    bc.plan(dims, brick, storage="fp8", src_dtype=src, max_w=16, max_h=16)
    bc.bind()
    bc.load(wide[:, :dims[1], ::stride])
    for b in rc.brick_grid(dims, brick):
        g = rc.ghosted_region(vol.astype(np.float32), b)
        buf, padded = bc.read_brick(b.index)
        arr = binding.unswizzle(buf, padded)
        tails, repeated = binding.row_tails(buf, padded)
        assert np.array_equal(tails, repeated)
        want = encoders.fp8_encode_brick(g, *encoders.brick_scale_offset(float(g.min()), float(g.max())))
        want = np.pad(want, [(0, p - n) for p, n in zip(arr.shape, want.shape)], mode="edge")
        assert np.array_equal(arr, want), b.index
    bc.close()
