"""The rule that chooses the fp32 dW kernel for few rows, on the CPU (a host function of the library)."""
import ctypes
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
    return lambda rows, cols, n, prefetch=0, masked=False, kept=0.1: f(0, rows, cols, n, prefetch, masked, kept)


def test_outputs_beyond_the_second_axis_of_a_grid(small_pays):
    """32 outputs a workgroup on an axis that holds 65535 of them: wider layers (up to 2^24 outputs are accepted) are the
    tile kernel's."""
    took = [(rows, cols, n, prefetch, masked, kept)
            for rows in (64, 128, 200, 250, 256) for cols in (1, 16, 32, 64, 784) for n in (65535 * 32 + 1, 3000000, 1 << 24)
            for prefetch in (0, 1, 2, 3) for masked in (False, True) for kept in (1e-6, 0.02, 0.1, 1.0)
            if small_pays(rows, cols, n, prefetch, masked, kept)]
    assert not took, took[:5]
