"""Autotuning keeps what it cannot tell apart: a frame of few samples has one
workgroup per work item, so its launch says nothing about the count of
persistent workgroups that later frames and captured ones are launched with."""
import numpy as np
import pytest

from gpu_util import gpu_render
from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


def _caster(size, brick, graph, step=0.5):
    rng = np.random.default_rng(3)
    vol = rng.standard_normal((60, 64, 56)).astype(np.float32)
    views = [synth.orbit_view(vol.shape[::-1], 5, kind="persp", width=size[0], height=size[1], step=step)]
    img, bc = gpu_render(vol, brick, views, synth.ramp_tf(-3, 4, lo=0.5), -3.0, 4.0, keep=True,
                         options={binding.BC_OPT_RENDER_WORKGROUPS: 777, binding.BC_OPT_GRAPH: graph})
    return img, bc


def test_small_frame_keeps_the_workgroup_count():
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    img, bc = _caster((48, 40), (32, 32, 32), 0)
    assert bc.stats()["n_tiles"] < 4 * 2 * n_cu          # fewer waves' worth of items than any candidate's
    chunk, wgs, tile_w = bc.autotune(frames=2)
    assert wgs == 777 and chunk in (32, 64) and tile_w in (4, 8, 16)
    assert np.abs(bc.render().cpu().numpy() - img).max() <= 1e-6
    bc.close()


@pytest.mark.parametrize("size,brick,graph,step", [((48, 40), (32, 32, 32), 1, 0.5), ((1400, 1050), (9, 9, 9), 0, 0.05)])
def test_persistent_launches_are_tuned(size, brick, graph, step):
    """Captured frames always take the persistent launch, and so do frames of
    many samples: the count comes from the candidates."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    img, bc = _caster(size, brick, graph, step)
    chunk, wgs, tile_w = bc.autotune(frames=2)
    assert wgs in [k * n_cu for k in (2, 4, 6, 8)] and chunk in (32, 64) and tile_w in (4, 8, 16)
    for _ in range(3):
        assert np.abs(bc.render().cpu().numpy() - img).max() <= 1e-6
    bc.close()
