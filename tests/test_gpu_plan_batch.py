"""The keep sets of all layers of a model, drawn together: more layers than one launch serves (8), widths that need different
kernels in one model, few and many rows (short rows share the kernel for longer ones up to 4096 of them)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import rad_oracle as R


@pytest.fixture(scope="module")
def ctx():
    from paper_2007_10412_amd import binding as B
    c = B.rad_ctx_create()
    yield c
    B.rad_ctx_destroy(c)


@pytest.mark.parametrize("batch,dims", [(5, (70, 300, 1100, 255, 9, 600, 1024, 64, 1025, 30, 4096, 3)), (1500, (130, 600, 40, 5)),
                                        (3, (8, 8))])
@pytest.mark.parametrize("scheme,p", [(1, 0.2), (2, 0.1), (3, 0.1), (4, 0.3), (5, 0.1)])
def test_columns_of_every_layer(ctx, batch, dims, scheme, p):
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, empty
    print("plan batch", batch, dims, scheme, flush=True)
    d = synth.mlp(seed=2, batch=batch, dims=dims)
    params, grads = [], []
    for W in d["Ws"]:
        params.append(dev(W)); grads.append(empty(W.shape))
    m = B.rad_model_create_mlp(ctx, B.RAD_F32, batch, list(dims), False, scheme, p)
    try:
        B.rad_train_step(ctx, m, B.make_sampling(scheme, p, 11, 40, 0), dev(d["x"]), dev(d["labels"]), params, grads)
        ref = R.mlp_train_step(d["x"], d["labels"], d["Ws"], None, scheme, p, 11, stream_base=40)
        for l in range(len(dims) - 1):
            rp, col, _ = B.rad_store_export_csr(ctx, B.rad_model_store(m, l), batch)
            assert np.array_equal(rp, ref["stores"][l][0]) and np.array_equal(col, ref["stores"][l][1]), l
    finally:
        B.rad_model_destroy(m)


@pytest.mark.parametrize("scheme", [1, 5])
def test_rows_of_all_layers_beyond_one_grid(ctx, scheme):
    """Four layers of 4.3 million rows, a workgroup of 256 threads each: together more threads than a grid may have.  The keep
    sets are those of stores that draw on their own."""
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import empty
    batch, dims, p = 4300000, (3, 4, 2, 3, 2), 0.5
    print("plan batch beyond a grid", scheme, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(1)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng)  # noqa: E731
    params = [r(a, b) for a, b in zip(dims, dims[1:])]
    grads, x = [empty(tuple(w.shape)) for w in params], r(batch, dims[0])
    labels = torch.randint(0, dims[-1], (batch,), device="cuda", dtype=torch.int32, generator=rng)
    m = B.rad_model_create_mlp(ctx, B.RAD_F32, batch, list(dims), False, scheme, p)
    try:
        B.rad_train_step(ctx, m, B.make_sampling(scheme, p, 11, 40, 0), x, labels, params, grads)
        for l in range(len(dims) - 1):
            rp, col, _ = B.rad_store_export_csr(ctx, B.rad_model_store(m, l), batch)
            st = B.rad_store_create(ctx, B.make_layer(batch, dims[l], dims[l + 1]), scheme, p)
            B.rad_sample_pack(ctx, B.make_sampling(scheme, p, 11, 40 + l, 0), torch.zeros(batch, dims[l], device="cuda"), st)
            want = B.rad_store_export_csr(ctx, st, batch)
            B.rad_store_destroy(st)
            assert np.array_equal(rp, want[0]) and np.array_equal(col, want[1]), l
    finally:
        B.rad_model_destroy(m)
