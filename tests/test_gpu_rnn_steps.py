"""The recurrent model with a launch per time step, for hidden states that elsewhere take a chunk of steps per launch: on a
stream kept to a part of the chip every model takes this route.  The gradients of a chunk of eight steps are formed on a
second stream; stores planned per step and the projections keep the step-by-step form."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_rnn import run_rnn
from tests.test_gpu_rnn_streams import assert_identical, step_twice
from tests.test_gpu_rnn_wide import data


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2007_10412_amd import binding as B
    torch.zeros(1, device="cuda")
    hip = ctypes.CDLL("libamdhip64.so")
    stream, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*([0x0fffffff] * 8))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    c = B.rad_ctx_create(torch.cuda.ExternalStream(stream.value))
    yield c
    torch.cuda.synchronize()
    assert B.rad_debug_redone_launches(c) == (0, 0)            # (no chunk of steps was launched)
    B.rad_ctx_destroy(c)
    assert hip.hipStreamDestroy(stream) == 0


@pytest.mark.parametrize("T", [1, 2, 10, 17])
@pytest.mark.parametrize("scheme,p", [(1, 0.3), (3, 0.25), (0, 1.0), (2, 0.25), (4, 0.25), (5, 0.25), (6, 0.25), (7, 0.25)])
def test_lengths_around_the_chunks(ctx, T, scheme, p):
    """T - 1 = 0: no recurrent gradient; 1: a single short chunk; 9: one whole chunk and one step; 16: two whole chunks."""
    run_rnn(ctx, data(20 + T, 8, T, 200, d_input=2, classes=5), scheme, p, seed=T, check_store=T > 1 and scheme < 6)


@pytest.mark.parametrize("batch,hidden,T", [(64, 576, 6), (20, 1024, 10), (130, 700, 3)])
def test_widths(ctx, batch, hidden, T):
    """576: split ranges of the products that have to be rounded to whole slices."""
    run_rnn(ctx, data(6, batch, T, hidden), 1, 0.2, seed=3)


def test_more_classes_than_hidden_units(ctx):
    run_rnn(ctx, data(264, 64, 4, 200, classes=500), 1, 0.5, seed=6)


@pytest.mark.parametrize("scheme", [1, 3, 5])
@pytest.mark.parametrize("T", [2, 3, 21])
def test_index_free_equals_indexed(ctx, scheme, T):
    """x~ of a chunk of time steps is rebuilt on the second stream from the keep bitmap of the step's own plan, or (T = 2, a
    store of one step) by drawing again; every step is taken twice with the same bits."""
    from tests.gpu_util import assert_grad_close
    d, res = data(40 + T, 24, T, 200), {}
    for mode in (False, True):
        a, b = step_twice(ctx, d, scheme, 0.2, seed=9, index_free=mode)
        assert_identical(a, b)
        res[mode] = a
    assert res[False][0] == res[True][0]
    for u, v in zip(res[False][2], res[True][2]):
        assert np.array_equal(u, v)
    for u, v in zip(res[True][1], res[False][1]):
        assert_grad_close(u, v, 1e-5, T * 24)
