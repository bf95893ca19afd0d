"""Layer calls recorded into a HIP graph by a context that has not run yet and so has no workspaces: the routes that want one
keep to those that do without.  Every replay, with new inputs each time, against the products in fp64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def captured(calls, stream):
    import torch
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        calls()
    return graph


@pytest.mark.parametrize("batch,d_in,d_out", [(300, 520, 263), (1000, 768, 3072), (2048, 4096, 40), (4096, 2048, 4096)])
def test_masked_layer(batch, d_in, d_out):
    """bf16 with ReLU: without a workspace the gradient is masked by the products' loaders."""
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import host, empty, assert_grad_close, U_F32, U_BF16
    print("capture", batch, d_in, d_out, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(batch + d_in + d_out)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16)  # noqa: E731
    x, W, dy = r(batch, d_in), r(d_in, d_out), r(batch, d_out)
    y, dX, dW = torch.empty_like(dy), torch.empty_like(x), empty((d_in, d_out))
    layer = B.make_layer(batch, d_in, d_out, dtype=B.RAD_BF16, relu=True)
    stream = torch.cuda.Stream()
    ctx = B.rad_ctx_create(stream)
    store = B.rad_store_create(ctx, layer, B.RAD_EXACT, 1.0)

    def calls():
        B.rad_forward_sample(ctx, layer, B.make_sampling(B.RAD_EXACT, 1.0, 1), x, W, None, y, store)
        B.rad_backward_dW(ctx, layer, store, dy, dW)
        B.rad_backward_dX(ctx, layer, store, dy, W, dX)
    try:
        graph = captured(calls, stream)
        for _ in range(3):
            x.copy_(r(batch, d_in)), dy.copy_(r(batch, d_out)), dW.fill_(float("nan")), dX.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            g = dy.double() * (y > 0)
            assert_grad_close(host(dW), (x.double().t().contiguous() @ g).cpu().numpy(), 1e-4, batch, "dW", acc_u=U_F32)
            assert_grad_close(host(dX), (g @ W.double().t().contiguous()).cpu().numpy(), 2e-2, d_out, "dX", acc_u=U_F32, out_u=2 * U_BF16)
    finally:
        graph = None
        B.rad_store_destroy(store)
        B.rad_ctx_destroy(ctx)


@pytest.mark.parametrize("dtype,batch,d_in,d_out,p", [(0, 1024, 2048, 1024, 0.5), (0, 300, 784, 10, 0.1), (1, 300, 784, 10, 0.05)])
def test_dW_from_the_store(dtype, batch, d_in, d_out, p):
    """dW whose rows would be split, with a workspace for the partial sums: recorded without one."""
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import host, empty, assert_grad_close, U_F32
    print("capture dW", dtype, batch, d_in, d_out, p, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(batch + d_in + d_out)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16 if dtype else torch.float32)  # noqa: E731
    x, dy, dW = r(batch, d_in), r(batch, d_out), empty((d_in, d_out))
    layer = B.make_layer(batch, d_in, d_out, dtype=dtype, relu=False)
    stream = torch.cuda.Stream()
    ctx = B.rad_ctx_create(stream)
    store = B.rad_store_create(ctx, layer, B.RAD_FIXEDK_PER_EXAMPLE, p)
    try:
        torch.cuda.synchronize()
        B.rad_sample_pack(ctx, B.make_sampling(B.RAD_FIXEDK_PER_EXAMPLE, p, 1), x, store)
        rp, col, val = B.rad_store_export_csr(ctx, store, batch)
        xs = torch.zeros(batch, d_in, device="cuda", dtype=torch.float64)
        rows = np.repeat(np.arange(batch), np.diff(rp))
        xs[torch.from_numpy(rows).cuda(), torch.from_numpy(col.astype(np.int64)).cuda()] = torch.from_numpy(val.astype(np.float64)).cuda()
        graph = captured(lambda: B.rad_backward_dW(ctx, layer, store, dy, dW), stream)
        for _ in range(3):
            dy.copy_(r(batch, d_out)), dW.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert_grad_close(host(dW), (xs.t().contiguous() @ dy.double()).cpu().numpy(), 1e-4, batch, "dW", acc_u=U_F32)
    finally:
        graph = None
        B.rad_store_destroy(store)
        B.rad_ctx_destroy(ctx)
