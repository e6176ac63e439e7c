"""The visibility order where its forms meet: a rank count up to 256 bricks, a
network in registers up to 1024, one in shared memory beyond; a single view and
four, from outside, from inside and with equal keys."""
import numpy as np
import pytest

from gpu_util import cam_of
from oracle import raycast as rc
from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 1, 1), (16, 16, 1), (257, 1, 1), (10, 10, 5), (9, 8, 12), (32, 32, 1),
                                  (41, 25, 1), (12, 12, 24)])
def test_order(dims):
    import torch
    bricks = rc.brick_grid(dims, (1, 1, 1))
    assert len(bricks) == dims[0] * dims[1] * dims[2]
    size = 24
    inside = synth.ViewSpec(synth.look_at((0.4 * dims[0], 0.6 * dims[1], 0.3 * dims[2]), (dims[0], 0.0, 0.0), (0.0, 1.0, 0.0)),
                            synth.perspective(60.0, 1.0, 0.1, 1000.0), size, size)
    views = [synth.orbit_view(dims, 11, kind="persp", width=size, height=size, elevation_deg=25.0), inside,
             synth.axis_view(dims, "z", dims[0], dims[1]),                       # whole planes of equal keys
             synth.orbit_view(dims, 3, kind="ortho", width=size, height=size, elevation_deg=-40.0)]
    views = [synth.ViewSpec(v.modelview, v.projection, size, size, 0.5, 0.99) for v in views]
    bc = binding.BrickCaster(0)
    bc.plan(dims, (1, 1, 1), max_views=4, max_w=size, max_h=size, max_tiles=4 * 9 * len(bricks))
    bc.bind()
    bc.load(torch.zeros(dims[::-1], device="cuda"))
    bc.set_transfer_function(synth.ramp_tf(-1.0, 1.0), -1.0, 1.0)
    want = [np.asarray(rc.visibility_order(bricks, cam_of(v))[0], np.int32) for v in views]
    for first, count in ((0, 4), (0, 1), (1, 1), (2, 1), (3, 1), (1, 2)):
        bc.set_views(views[first:first + count])
        bc.render()
        for v in range(count):
            assert np.array_equal(bc.visibility_order(v), want[first + v]), (first, count, v)
    bc.close()
