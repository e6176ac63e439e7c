"""Views on both sides of the distance from which rays start beside the cube
instead of at the eye, in one launch, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import raycast as rc
from paper_1205_0282_amd import binding, synth

from gpu_util import TOL, cam_of, compare, gpu_render

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [32, 64])
@pytest.mark.parametrize("kind,skew", [("persp", 0.0), ("persp", 0.4), ("ortho", 0.0)])
def test_near_and_far_eyes(kind, skew, chunk):
    """Eyes 3.9 and 4.1 half-diagonals from the centre (the line is at 4), 115 and
    2,300 half-diagonals away; skewed: the cube beside the image's centre."""
    rng = np.random.default_rng(5)
    dims, brick, step = (37, 29, 23), (12, 13, 9), 0.43
    vol = rng.uniform(-1, 1, dims[::-1]).astype(np.float32)
    rgba = synth.random_tf(rng, 16, alpha_max=0.6)
    views = []
    for k, fovy in enumerate((29.8, 28.2, 1.0, 0.05)):
        v = synth.orbit_view(dims, 5 + 16 * k, kind=kind, width=44, height=36, fovy_deg=fovy, step=step, ert=0.97)
        p = np.array(v.projection, np.float64).reshape(16)
        p[8] += skew
        views.append(synth.ViewSpec(v.modelview, p, v.width, v.height, v.step, v.ert))
    img, bc = gpu_render(vol, brick, views, rgba, -1.0, 1.0, keep=True,
                         options={binding.BC_OPT_SAMPLE_CHUNK: chunk})
    tf = rc.TransferFunction(rgba, -1.0, 1.0)
    stored = rc.store_bricks(vol, rc.brick_grid(dims, brick))
    for i, v in enumerate(views):
        res = rc.render_bricked(stored, dims, cam_of(v), tf, step, 0.97)
        err, n_tie, n_ovf = compare(img[i].reshape(-1, 4), res, f"view {i}")
        assert err <= TOL, (i, err)
        assert res.image[:, 3].max() > 0.5
    bc.close()
