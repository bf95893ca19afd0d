"""The rule that chooses the fp32 dW kernel for few rows, on the CPU (a host function of the library)."""
import ctypes
import math
import os

import pytest


@pytest.fixture(scope="module")
def small_pays():
    from paper_2007_10412_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    f = getattr(binding.lib(), "_ZN3rad13dw_small_paysEiiiiibd")     # rad::dw_small_pays
    f.restype = ctypes.c_bool
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_bool, ctypes.c_double]
    return lambda *call: f(0, *call)


def test_outputs_beyond_the_second_axis_of_a_grid(small_pays):
    """32 outputs a workgroup on an axis that holds 65535 of them: wider layers (up to 2^24 outputs are accepted) are the
    tile kernel's."""
    took = [(rows, cols, n, prefetch, masked, kept)
            for rows in (64, 128, 200, 250, 256) for cols in (1, 16, 32, 64, 784) for n in (65535 * 32 + 1, 3000000, 1 << 24)
            for prefetch in (0, 1, 2, 3) for masked in (False, True) for kept in (1e-6, 0.02, 0.1, 1.0)
            if small_pays(rows, cols, n, prefetch, masked, kept)]
    assert not took, took[:5]


# fraction, masked, us of the other side (tiles or row split) and of the one-pass kernel
@pytest.mark.parametrize("rows,cols,n,kept,masked,other,here", [
    (145, 3087, 90, 0.8, True, 21.8, 29.4), (235, 230, 2396, 0.6, False, 25.8, 34.0), (225, 3332, 125, 0.8, True, 31.0, 39.0),
    (105, 141, 3927, 0.25, True, 16.4, 19.7), (123, 110, 3792, 0.25, True, 11.5, 13.6), (123, 2893, 198, 0.15, True, 18.1, 20.4),
    (150, 2048, 1024, 0.1, False, 15.7, 25.4),
    (256, 1024, 1024, 0.1, False, 17.9, 14.5), (256, 512, 2048, 0.1, False, 17.9, 13.6), (150, 784, 300, 0.1, False, 11.8, 5.5),
    (150, 300, 300, 0.1, False, 11.7, 5.2)])
def test_the_faster_side(small_pays, rows, cols, n, kept, masked, other, here):
    mean = kept * min(cols, 256)
    prefetch = math.ceil((mean + 6.0 * math.sqrt(mean)) / 16)
    assert small_pays(rows, cols, n, prefetch, masked, kept) == (here < other)
