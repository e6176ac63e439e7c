"""The small oracle tests on the persistent ray caster.  Frames of few samples
take the launch with four lanes to a ray, so the parity tests' small frames no
longer reach the persistent kernel with 32-sample chunks; captured frames
always do.  Every check is the parity test's own, with its frames captured."""
import pytest

import gpu_util
import test_gpu_mip as mip_tests
import test_gpu_parity as parity
from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cube():
    return synth.make_cube(synth.RECIPE_SMALL, workers=4)


@pytest.fixture(autouse=True)
def captured(monkeypatch):
    def render(*args, options=None, **kw):
        return gpu_util.gpu_render(*args, options={**(options or {}), binding.BC_OPT_GRAPH: 1}, **kw)
    monkeypatch.setattr(parity, "gpu_render", render)
    monkeypatch.setattr(mip_tests, "gpu_render", render)


@pytest.mark.parametrize("tau", [1.0, 0.99])
def test_small_plain_full_frame(cube, tau):
    parity.test_small_plain_full_frame(cube, tau)


@pytest.mark.parametrize("n,brick,kind,seed", [(8, (3, 5, 2), "persp", 1), (16, (16, 4, 9), "ortho", 4)])
def test_brute_force_cubes_four_views(n, brick, kind, seed):
    parity.test_brute_force_cubes_four_views(n, brick, kind, seed)


@pytest.mark.parametrize("storage", ["f16", "fp8"])
def test_precision_forms(cube, storage):
    parity.test_precision_forms_match_oracle_on_stored_values(cube, storage)


@pytest.mark.parametrize("K,kind", [(2, "random"), (1024, "ramp"), (1025, "ramp"), (4096, "ramp")])
def test_table_sizes(cube, K, kind):
    parity.test_table_sizes_at_the_limits(cube, K, kind)


@pytest.mark.parametrize("eye,target", [((70.3, 61.7, 45.2), (20.0, 90.0, 120.0)), ((64.0, 64.0, 64.0), (128.0, 20.0, 10.0)),
                                        ((30.5, 140.0, 64.2), (64.0, 0.0, 64.0))])
def test_eye_inside_or_next_to_the_cube(cube, eye, target):
    parity.test_eye_inside_or_next_to_the_cube(cube, eye, target)


@pytest.mark.parametrize("step,brick,size", [(0.05, (20, 18, 22), (32, 24)), (3.3, (6, 6, 6), (44, 36)), (7.9, (6, 6, 6), (44, 36))])
def test_steps(step, brick, size):
    parity.test_steps_far_below_a_voxel_and_above_a_brick(step, brick, size)


@pytest.mark.parametrize("dims,brick", [((1, 1, 1), (1, 1, 1)), ((2, 1, 3), (1, 1, 2)), ((5, 1, 1), (2, 1, 1)),
                                        ((3, 4, 1), (3, 4, 1))])
def test_smallest_cubes(dims, brick):
    parity.test_smallest_cubes_bricks_and_frames(dims, brick)


def test_constructed_ties():
    parity.test_constructed_exact_ties_match_an_enumerated_result()


def test_fp8_decode():
    parity.test_fp8_decode_of_every_code()


@pytest.mark.parametrize("storage", ["f32", "fp8"])
def test_empty_space_skipping(cube, storage):
    parity.test_empty_space_skipping_is_bit_identical(cube, storage)


def test_hundred_bricks():
    parity.test_between_64_and_128_bricks()


@pytest.mark.parametrize("kind", ["persp", "ortho"])
def test_thin_edge_bricks(kind):
    parity.test_thin_edge_bricks_like_table1_shapes(kind)


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("kind,step", [("ortho", 0.5), ("persp", "voxel"), ("ortho", "voxel")])
def test_projection(cube, storage, kind, step):
    mip_tests.test_small_cube_matches_oracle(cube, storage, kind, step)


def test_projected_rays_stop_at_the_brick_maximum():
    mip_tests.test_rays_stop_at_the_brick_maximum()
