"""Four lanes to a ray against the persistent launch at the edges of the route:
frames just inside it and just outside, per-voxel projection that takes it for
its rays' spacing, and a learned frame whose coarse and validation passes both
take it side by side.  Images and sample counts are the same, bit for bit; which
launch a frame took is read from the profiler."""
import numpy as np
import pytest

from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


def _kernels(frame):
    """Names of the ray-casting kernels that frame() launches."""
    import torch
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        frame()
        torch.cuda.synchronize()
    return [k for k in ("render_quad_kernel", "render_kernel") for e in p.key_averages() if k in e.key for _ in range(e.count)]


def _caster(dims, brick, storage, size, views=1):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(dims[0])
    bc = binding.BrickCaster(0)
    bc.plan(dims, (brick,) * 3, storage=storage, max_views=views, max_w=size[0], max_h=size[1], max_tiles=1 << 18)
    bc.bind()
    bc.load(torch.randn(dims[::-1], generator=g, device="cuda"))
    bc.set_transfer_function(synth.ramp_tf(-5.0, 5.0, lo=1.0), -5.0, 5.0)
    return bc


def _same_as_persistent(bc, quads):
    """Renders with the route's launch and, captured, with the persistent one."""
    import torch
    got = []
    for graph in (0, 1):
        bc.set_option(binding.BC_OPT_GRAPH, graph)
        img = bc.render().clone()
        torch.cuda.synchronize()
        st = bc.stats()
        got.append((img, st["nominal_samples"], st["evaluated_samples"], st["n_tiles"]))
    bc.set_option(binding.BC_OPT_GRAPH, 0)
    assert torch.equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:] and got[0][2] > 0
    names = set(_kernels(bc.render))
    assert names == {"render_quad_kernel" if quads else "render_kernel"}, names


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("dims,brick,size,step,quads", [
    ((64, 64, 64), 32, (1280, 720), 0.5, True), ((64, 64, 64), 32, (1920, 1080), 0.125, False),
    ((60, 70, 50), 16, (800, 600), 0.5, True), ((60, 70, 50), 16, (1920, 1080), 0.5, False),
    ((96, 96, 96), 96, (1920, 1080), 1.0, True), ((96, 96, 96), 96, (1920, 1080), 0.125, False)])
def test_about_the_line(storage, dims, brick, size, step, quads):
    bc = _caster(dims, brick, storage, size)
    bc.set_views([synth.orbit_view(dims, 7, width=size[0], height=size[1], elevation_deg=15.0, step=step)])
    _same_as_persistent(bc, quads)
    bc.close()


@pytest.mark.parametrize("storage,zoom,quads", [("f32", 1.0, True), ("f16", 1.0, True), ("fp8", 1.0, False),
                                                ("f32", 3.0, False), ("f16", 3.0, False)])
def test_per_voxel_projection(storage, zoom, quads):
    """Some 30 K items of 256 samples a ray, with 2 voxels between rays: too many
    for the samples' estimate alone."""
    dims, size = (1100, 1100, 700), (860, 860)
    bc = _caster(dims, 256, storage, size)
    bc.set_operator("mip", "voxel")
    v = synth.orbit_view(dims, 7, width=size[0], height=size[1], elevation_deg=15.0)
    p = np.array(v.projection, np.float64).reshape(16)
    p[0] *= zoom
    p[5] *= zoom
    bc.set_views([synth.ViewSpec(v.modelview, p, v.width, v.height, v.step, v.ert)])
    _same_as_persistent(bc, quads)
    bc.close()


def test_learned_passes_side_by_side():
    """Coarse and validation passes together, each with four lanes to a ray,
    against the same frame captured (both persistent)."""
    import torch
    from oracle import cnn
    dims, size = (128, 120, 110), (320, 240)
    for threshold in (-1e9, 1e9):                          # passes; falls back
        got = []
        for graph in (0, 1):
            bc = _caster(dims, 64, "f32", size, views=2)    # (the validation tiles follow the frame's number)
            bc.cnn_setup(2, size[1] // 2, size[0] // 2)
            bc.cnn_set_weights(cnn.init_params(21))
            bc.set_option(binding.BC_OPT_GRAPH, graph)
            bc.set_learned(True, coarse_step=2.0, psnr_threshold_db=threshold, validate_stride=4)
            bc.set_views([synth.orbit_view(dims, f, width=size[0], height=size[1]) for f in (3, 30)])
            img = bc.render().clone()
            torch.cuda.synchronize()
            got.append((img, bc.stats()))
            if not graph:
                names = _kernels(bc.render)
                assert names.count("render_quad_kernel") == 2, names
            bc.close()
        assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
        assert got[0][1]["fell_back"] == (1 if threshold > 0 else 0)
