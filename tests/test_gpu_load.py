"""Brick loading at the sizes where its kernels change: stored rows from one
micro-block to the widest brick (whose staged rows pass 64 KiB), sources with
strides, and values that min/max must pass by."""
import numpy as np
import pytest

from oracle import encoders
from oracle import raycast as rc
from paper_1205_0282_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("dims,brick,stride", [((1030, 5, 3), (1024, 8, 8), 1), ((62, 7, 6), (64, 4, 4), 1),
                                               ((1, 1, 1), (4, 4, 4), 1), ((67, 9, 5), (63, 3, 5), 3)])
def test_stored_rows(storage, dims, brick, stride):
    import torch
    rng = np.random.default_rng(21)
    vol = rng.standard_normal(dims[::-1]).astype(np.float32)
    src = torch.full((dims[2], dims[1] + 1, stride * dims[0]), 1e9, device="cuda")
    src[:, :dims[1], ::stride] = torch.from_numpy(vol).cuda()
    bc = binding.BrickCaster(0)
    bc.plan(dims, brick, storage=storage, max_w=16, max_h=16)
    bc.bind()
    bc.load(src[:, :dims[1], ::stride])
    _, so, mm = bc.bricks()
    for b in rc.brick_grid(dims, brick):
        g = rc.ghosted_region(vol, b)
        buf, padded = bc.read_brick(b.index)
        arr = binding.unswizzle(buf, padded)
        tails, repeated = binding.row_tails(buf, padded)
        assert np.array_equal(tails, repeated)
        # the padding repeats the last ghost
        g = np.pad(g, [(0, p - n) for p, n in zip(arr.shape, g.shape)], mode="edge")
        assert mm[b.index, 0] == g.min() and mm[b.index, 1] == g.max()
        if storage == "f32":
            want = g
        elif storage == "f16":
            want = encoders.f16_bits(g)
        else:
            want = encoders.fp8_encode_brick(g, *encoders.brick_scale_offset(float(g.min()), float(g.max())))
        assert np.array_equal(arr, want)
    bc.close()


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
def test_minmax_passes_nan_by(storage):
    import torch
    vol = np.random.default_rng(22).standard_normal((9, 11, 70)).astype(np.float32)
    vol[4, 5, 33] = np.nan
    vol[0, 0, 0] = np.nan
    bc = binding.BrickCaster(0)
    bc.plan(vol.shape[::-1], (40, 6, 9), storage=storage, max_w=16, max_h=16)
    bc.bind()
    bc.load(torch.from_numpy(vol).cuda())
    _, _, mm = bc.bricks()
    for b in rc.brick_grid(vol.shape[::-1], (40, 6, 9)):
        g = rc.ghosted_region(vol, b)
        assert mm[b.index, 0] == np.nanmin(g) and mm[b.index, 1] == np.nanmax(g)
    bc.close()


@pytest.mark.parametrize("storage,stride", [("f32", 1), ("fp8", 2)])
def test_host_source_gathered_by_threads(storage, stride):
    """A host source large enough for several threads, in ragged bricks and
    more of them than staging buffers, stores what a device source stores."""
    import torch
    rng = np.random.default_rng(23)
    vol = rng.standard_normal((70, 130, 151)).astype(np.float32)
    wide = np.full((70, 131, 151 * stride), 1e9, np.float32)
    wide[:, :130, ::stride] = vol
    pools = []
    for source in (torch.from_numpy(vol).cuda(), wide[:, :130, ::stride]):
        bc = binding.BrickCaster(0)
        bc.plan(vol.shape[::-1], (64, 47, 33), storage=storage, max_w=16, max_h=16)
        bc.bind()
        for _ in range(2):
            bc.load(source)
        _, so, mm = bc.bricks()
        pools.append([so, mm] + [bc.read_brick(b)[0] for b in range(len(mm))])
        bc.close()
    for a, b in zip(*pools):
        assert np.array_equal(a, b)
