"""Frames of few work items take the ray caster with four lanes to a ray; a
captured frame always takes the persistent one.  Both must give the same bits
and the same sample counts, for every form that the frame can have."""
import numpy as np
import pytest

from gpu_util import gpu_render
from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,src", [("f32", np.float32), ("f16", np.float16), ("fp8", np.float32)])
@pytest.mark.parametrize("op,K,step,ert,options", [
    (("composite", "fixed"), 256, 0.5, 0.99, {}),
    (("composite", "fixed"), 2, 0.37, 0.3, {binding.BC_OPT_EMPTY_SKIP: 0}),
    (("composite", "fixed"), 1025, 1.3, 1.0, {binding.BC_OPT_TILE_WIDTH: 16, binding.BC_OPT_XCD_QUEUES: 0}),
    (("composite", "fixed"), 1024, 0.05, 0.9, {binding.BC_OPT_TILE_WIDTH: 4}),
    (("mip", "fixed"), 300, 0.5, 1.0, {}),
    (("mip", "voxel"), 64, 0.5, 1.0, {binding.BC_OPT_EMPTY_SKIP: 0, binding.BC_OPT_TILE_WIDTH: 4}),
])
def test_same_bits_as_the_persistent_launch(storage, src, op, K, step, ert, options):
    rng = np.random.default_rng(K)
    vol = rng.standard_normal((33, 41, 58)).astype(src)
    tf = synth.random_tf(rng, K, 0.3)
    if op[0] == "composite":
        tf[rng.uniform(size=K) < 0.6, 3] = 0.0
    else:
        tf[: K // 2] = tf[0]
    dims = vol.shape[::-1]
    views = [synth.orbit_view(dims, fr, kind="persp", width=75, height=53, elevation_deg=el, step=step, ert=ert)
             for fr, el in ((0, 0.0), (9, 35.0), (31, -50.0))]
    got = []
    for graph in (0, 1):
        img, bc = gpu_render(vol, (19, 41, 12), views, tf, -2.0, 2.5, storage=storage, op=op, keep=True,
                             options={**options, binding.BC_OPT_GRAPH: graph})
        st = bc.stats()
        got.append((img, st["nominal_samples"], st["evaluated_samples"], st["n_tiles"]))
        bc.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert got[0][1:] == got[1][1:] and got[0][2] > 0


def test_counts_start_over_with_each_frame():
    """The persistent launch and the one with a workgroup per item keep their
    sample counts in different places: a frame shows its own only."""
    rng = np.random.default_rng(5)
    vol = rng.standard_normal((20, 24, 28)).astype(np.float32)
    view = synth.orbit_view(vol.shape[::-1], 3, width=40, height=32)
    _, bc = gpu_render(vol, (16, 16, 16), [view], synth.ramp_tf(-3, 4, lo=0.5), -3.0, 4.0, keep=True)
    first = bc.stats()
    for graph in (1, 0, 0, 1):
        bc.set_option(binding.BC_OPT_GRAPH, graph)
        bc.render()
        assert bc.stats() | {"psnr_db": 0} == first | {"psnr_db": 0}
    bc.close()
