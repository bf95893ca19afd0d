"""dW of a bf16 layer from its store where two groups of threads take half of the batch each: batches around the slices of 32
rows and their halves, outputs around the tile of 256 x 64 and the number of tiles a chip holds (256)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2007_10412_amd import binding as B
    c = B.rad_ctx_create()
    yield c
    B.rad_ctx_destroy(c)


@pytest.mark.parametrize("batch", [127, 128, 129, 159, 160, 161, 193, 800])
@pytest.mark.parametrize("d_in,d_out", [(100, 16), (256, 64), (300, 72), (513, 130), (4096, 1024), (4096, 1030)])
@pytest.mark.parametrize("scheme,p", [(1, 0.1), (3, 0.03)])
@pytest.mark.parametrize("relu", [False, True])
def test_dW(ctx, batch, d_in, d_out, scheme, p, relu):
    import numpy as np
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import empty, host, assert_grad_close, U_F32
    print("dW halves", batch, d_in, d_out, scheme, relu, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(batch + d_in + d_out)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16)  # noqa: E731
    x, W, dy = r(batch, d_in), r(d_in, d_out), r(batch, d_out)
    y, dW = torch.empty_like(dy), empty((d_in, d_out))
    layer = B.make_layer(batch, d_in, d_out, dtype=B.RAD_BF16, relu=relu)
    store = B.rad_store_create(ctx, layer, scheme, p)
    try:
        B.rad_forward_sample(ctx, layer, B.make_sampling(scheme, p, 7, 0, 0), x, W, None, y, store)
        B.rad_backward_dW(ctx, layer, store, dy, dW)
        rp, col, val = B.rad_store_export_csr(ctx, store, batch)
    finally:
        B.rad_store_destroy(store)
    xs = np.zeros((batch, d_in))
    xs[np.repeat(np.arange(batch), np.diff(rp)), col] = val
    f = lambda t: t.double().cpu().numpy()  # noqa: E731
    g = f(dy) * (f(y) > 0) if relu else f(dy)
    assert_grad_close(host(dW), xs.T @ g, 1e-4, batch, "dW", acc_u=U_F32)
