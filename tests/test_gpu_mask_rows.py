"""bf16 layers with ReLU whose upstream gradient is masked in a pass of its own: output widths around the padding of its rows
(64 columns), its 16-byte chunks, and the width from which the pass is used (256)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2007_10412_amd import binding as B
    c = B.rad_ctx_create()
    yield c
    B.rad_ctx_destroy(c)


@pytest.mark.parametrize("d_out", [255, 256, 257, 263, 264, 319, 320, 512, 521])
@pytest.mark.parametrize("batch,d_in", [(1, 130), (70, 512), (1030, 511), (1030, 520)])
@pytest.mark.parametrize("bias", [False, True])
def test_masked_backward(ctx, batch, d_in, d_out, bias):
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import empty, host, assert_grad_close, U_F32
    print("mask rows", batch, d_in, d_out, bias, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(batch + d_in + d_out)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16)  # noqa: E731
    x, W, dy, b = r(batch, d_in), r(d_in, d_out), r(batch, d_out), (r(d_out).float() if bias else None)
    y, dX = torch.empty_like(dy), torch.empty_like(x)
    dW, db = empty((d_in, d_out)), empty((d_out,)) if bias else None
    layer = B.make_layer(batch, d_in, d_out, dtype=B.RAD_BF16, relu=True, has_bias=bias)
    store = B.rad_store_create(ctx, layer, B.RAD_EXACT, 1.0)
    B.rad_ctx_timing(ctx, "mask_rows")
    B.rad_ctx_timing_reset(ctx)
    try:
        B.rad_forward_sample(ctx, layer, B.make_sampling(B.RAD_EXACT, 1.0, 1, 0, 0), x, W, b, y, store)
        B.rad_backward_dW(ctx, layer, store, dy, dW, db)
        B.rad_backward_dX(ctx, layer, store, dy, W, dX)
        passes = B.rad_ctx_timing_read(ctx, "mask_rows")[0]
    finally:
        B.rad_ctx_timing(ctx, "")
        B.rad_store_destroy(store)
    used = d_out >= 256 and (d_in >= 512 or batch <= 1024)
    assert passes == (0 if not used else 1 if bias and d_out == 512 else 2)    # (512 wide: the bias sums write g on the way)
    f = lambda t: t.double().cpu().numpy()  # noqa: E731
    g = f(dy) * (f(y) > 0)
    assert_grad_close(host(dW), f(x).T @ g, 1e-4, batch, "dW", acc_u=U_F32)
    assert_grad_close(f(dX), g @ f(W).T, 2e-2, d_out, "dX", acc_u=U_F32, out_u=2.0 ** -8)
    if bias:
        assert_grad_close(host(db), g.sum(0), 1e-4, batch, "db", acc_u=U_F32)
