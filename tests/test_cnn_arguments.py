"""Argument checks of the upsampler's entry points that come before anything
touches a device: null and misaligned images."""
import ctypes as C

import pytest

from paper_1205_0282_amd import binding


@pytest.fixture
def ctx(lib):
    h = C.c_void_p()
    assert lib.bc_create(-1, C.byref(h)) == binding.BC_OK
    yield h
    lib.bc_destroy(h)


@pytest.mark.parametrize("entry", ["forward", "gradients", "train_step"])
@pytest.mark.parametrize("first,second,code", [(0, 256, binding.BC_E_ARG), (256, 0, binding.BC_E_ARG),
                                               (260, 512, binding.BC_E_ARG), (256, 520, binding.BC_E_ARG),
                                               (256, 512, binding.BC_E_STATE)])
def test_images(lib, ctx, entry, first, second, code):
    """The kernels read whole pixels, 16 bytes at a time."""
    a, b = C.c_void_p(first), C.c_void_p(second)
    if entry == "forward":
        got = lib.bc_cnn_forward(ctx, a, b, 1, 8, 8, None)
    elif entry == "gradients":
        got = lib.bc_cnn_gradients(ctx, a, b, 1, 8, 8, None, None)
    else:
        got = lib.bc_cnn_train_step(ctx, a, b, 1, 8, 8, 1e-3, None, None)
    assert got == code
