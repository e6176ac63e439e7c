"""Which launch a frame's ray casting takes: four lanes to a ray where that is
the faster one.  The persistent launch with 64-sample chunks, which no rule
takes away from, stands for the other choice; the shapes are those at which the
wrong one takes half as long again and more."""
import statistics

import numpy as np
import pytest

from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


def _ms(bc, out, chunk):
    bc.set_option(binding.BC_OPT_SAMPLE_CHUNK, chunk)
    for _ in range(2):
        bc.render(out)
    bc.enable_timing(True, stages=False)
    for _ in range(15):
        bc.render(out)
    t = statistics.median(bc.frame_times())
    bc.enable_timing(False)
    return t


@pytest.mark.parametrize("edge,brick,storage,op,size,zoom,step,low,high", [
    (64, 16, "f32", ("composite", "fixed"), (1920, 1080), 3.0, 1.0, 0.5, 1.3),     # many items of few samples
    (64, 16, "fp8", ("composite", "fixed"), (1024, 768), 3.0, 2.0, 0.5, 1.3),
    (512, 256, "f32", ("mip", "voxel"), (1920, 1080), 4.0, 0.5, 0.5, 1.2),         # a close view
    (512, 256, "f16", ("mip", "voxel"), (1920, 1080), 4.0, 0.5, 0.5, 1.2),
    (128, 64, "f32", ("composite", "fixed"), (256, 256), 1.0, 0.5, 0.0, 0.9),     # few items: the quads
    (96, 96, "f32", ("composite", "fixed"), (1920, 1080), 3.0, 2.0, 0.0, 0.9),    # one brick, one queue
])
def test_faster_launch(edge, brick, storage, op, size, zoom, step, low, high):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(edge)
    bc = binding.BrickCaster(0)
    bc.plan((edge,) * 3, (brick,) * 3, storage=storage, max_w=size[0], max_h=size[1], max_tiles=1 << 19)
    bc.bind()
    bc.load(torch.randn((edge,) * 3, generator=g, device="cuda"))
    bc.set_operator(*op)
    bc.set_transfer_function(synth.ramp_tf(-5.0, 5.0, lo=1.5), -5.0, 5.0)
    v = synth.orbit_view((edge,) * 3, 3, width=size[0], height=size[1], step=step)
    p = np.array(v.projection, np.float64).reshape(16)
    p[0] *= zoom
    p[5] *= zoom
    bc.set_views([synth.ViewSpec(v.modelview, p, v.width, v.height, v.step, v.ert)])
    out = torch.empty((1, size[1], size[0], 4), device="cuda")
    a, b = _ms(bc, out, 32), _ms(bc, out, 64)
    bc.close()
    print(f"{a * 1e3:.1f} us, persistent with 64-sample chunks {b * 1e3:.1f} us")
    assert low <= a / b <= high
