"""bench.py's account of the ray-casting kernel: the name of the one that ran, and
counter-measured traffic tied to the sources that choose it."""
from test_bench_cli import _bench_module


def test_traffic_is_tied_to_the_host_code_that_picks_the_kernel():
    assert "bc_api.cpp" in _bench_module().KERNEL_SOURCES


def test_kernel_by_name():
    bench = _bench_module()
    quad = "void (anonymous namespace)::render_quad_kernel<0, true, 0>(BcFramePtrs)"
    persistent = "void (anonymous namespace)::render_kernel<0, true, 32, 0, true>(BcFramePtrs)"
    others = ["hipLaunchKernel", "(anonymous namespace)::setup_kernel(BcFramePtrs)"]
    assert bench.ray_casting_kernel(others + [quad]) == "render_quad_kernel"
    assert bench.ray_casting_kernel([persistent] + others) == "render_kernel"
    assert bench.ray_casting_kernel(others) is None and bench.ray_casting_kernel([quad, persistent]) is None
