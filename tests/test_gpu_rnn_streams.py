"""The recurrent model with a launch per time step (hidden states above 192 with batches above 192): per-chunk gradients on
the side stream while the main stream goes on with the chain of dX products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_rnn import ctx, run_rnn  # noqa: F401

NAMES = ["W_ih", "W_hh", "b", "W_ho", "b_o"]


def step_twice(ctx, d, scheme, p, seed, index_free=False):  # noqa: F811
    """Loss, gradients and recurrent store of one step taken twice, another draw in between."""
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty
    Bt, T, I = d["x"].shape
    H, C = d["W_ho"].shape
    m = B.rad_model_create_rnn(ctx, Bt, T, I, H, C, scheme, p)
    try:
        if index_free:
            B.rad_model_set_index_free(ctx, m, True)
        params, grads = [dev(d[n]) for n in NAMES], [empty(d[n].shape) for n in NAMES]
        x, labels = dev(d["x"]), dev(d["labels"])
        runs = []
        for s in (seed, seed + 1, seed):
            for g in grads:
                g.fill_(float("nan"))
            loss = B.rad_train_step(ctx, m, B.make_sampling(scheme, p, s, 20, 0), x, labels, params, grads)
            store = B.rad_store_export_csr(ctx, B.rad_model_store(m, 0), (T - 1) * Bt) if scheme else ()
            runs.append((loss, [host(g).copy() for g in grads], store))
        return runs[0], runs[2]
    finally:
        B.rad_model_destroy(m)


def assert_identical(a, b):
    assert a[0] == b[0]
    for n, u, v in zip(NAMES, a[1], b[1]):
        assert np.isfinite(u).all() and np.array_equal(u.view(np.uint32), v.view(np.uint32)), n
    for u, v in zip(a[2], b[2]):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("scheme", [1, 3])
@pytest.mark.parametrize("batch,hidden,T,seed", [(256, 600, 10, 53), (256, 600, 18, 192), (320, 520, 2, 29), (320, 520, 10, 80)])
def test_split_sums_of_both_streams(ctx, batch, hidden, T, seed, scheme):  # noqa: F811
    """A first chunk of one step ((T - 2) % 8 == 0) whose dW splits its rows, beside a dX that splits K: both keep partial
    sums in a workspace at the same time, so each stream has to have one of its own.  Parity and two identical runs.
    (Seeds without a pre-activation within 2e-6 of its rms of zero: fp32 sums of 600 terms err by about 3e-7, and a ReLU
    that falls the other way moves a column of dW_hh by more than the bound.)"""
    from paper_2007_10412_amd import binding as B, synth
    d = synth.rnn(seed=seed, batch=batch, T=T, d_input=1, hidden=hidden, classes=10, identity=False)
    print("rnn streams", batch, hidden, T, scheme, flush=True)
    for kernel, least in (("dw_narrow", 2), ("splitk_reduce", T)):       # the route this is about: W_ho's dW, the first
        B.rad_ctx_timing(ctx, kernel)                                    # chunk's; their reductions and T - 2 or more of dX
        B.rad_ctx_timing_reset(ctx)
        try:
            runs = step_twice(ctx, d, scheme, 0.3, seed=9)
            assert B.rad_ctx_timing_read(ctx, kernel)[0] >= 3 * least
        finally:
            B.rad_ctx_timing(ctx, "")
            B.rad_ctx_timing_reset(ctx)
        assert_identical(*runs)
    assert_identical(*step_twice(ctx, d, scheme, 0.3, seed=9))
    run_rnn(ctx, d, scheme, 0.3, seed=9)
