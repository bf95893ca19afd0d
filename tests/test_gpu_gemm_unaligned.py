"""GPU parity of the bf16 GEMMs whose rows start at any element: widths and batches that are multiples of nothing, so
that 16-byte loads and stores are aligned to an element only, chunks run past the end of a row and the last slices are
guarded.  The three calls of one layer with ReLU (bits as loader masks, or, from 256 outputs on with 512 inputs or 1024
rows, a gradient masked ahead of the products) and of a layer without, against the oracle, at contraction lengths that end
the pipeline at every point; then the shapes whose wide tiles mask in their loaders."""
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


# (batch, d_in, d_out): below one chunk, around one slice of 32, around tiles of 128 and 256, long contractions; the
# last ones take the 256-wide tiles
@pytest.mark.parametrize("n,d,o", [(1, 1, 1), (3, 2, 5), (7, 9, 3), (33, 31, 10), (129, 65, 127), (40, 257, 130),
                                   (131, 289, 259), (300, 1101, 333), (1000, 331, 2050), (257, 4099, 2047),
                                   (2049, 2061, 4101)])
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("scheme", ["exact", "per_example"])
def test_layer_of_any_width(ctx, n, d, o, relu, scheme):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty, unpack_bits, assert_grad_close, TOL, U_BF16
    import torch
    sch, p = (B.RAD_EXACT, 1.0) if scheme == "exact" else (B.RAD_FIXEDK_PER_EXAMPLE, 0.2)
    if n * d * o > 10 ** 10 and scheme == "exact" and not relu:
        pytest.skip("the large shape once per mask and scheme is enough")
    rng = np.random.default_rng(n + 7 * d + 13 * o)
    x = R.round_bf16(rng.standard_normal((n, d)).astype(np.float32))
    W = R.round_bf16((rng.standard_normal((d, o)) / np.sqrt(d)).astype(np.float32))
    dy = R.round_bf16(rng.standard_normal((n, o)).astype(np.float32))
    print("layer", n, d, o, relu, scheme, flush=True)
    L = B.make_layer(n, d, o, dtype=B.RAD_BF16, relu=relu)
    st = B.rad_store_create(ctx, L, sch, p)
    try:
        y, dW, dX = empty((n, o), B.RAD_BF16), empty((d, o)), empty((n, d), B.RAD_BF16)
        xd, Wd, dyd = dev(x, B.RAD_BF16), dev(W, B.RAD_BF16), dev(dy, B.RAD_BF16)
        B.rad_forward_sample(ctx, L, B.make_sampling(sch, p, 5), xd, Wd, None, y, st)
        h = (xd.double() @ Wd.double()).cpu().numpy()
        want = np.maximum(h, 0) if relu else h
        assert_grad_close(host(y), want, TOL[B.RAD_BF16], d, "y", out_u=2 * U_BF16)
        g = dy
        if relu:
            bits = unpack_bits(B.rad_store_export_bits(ctx, st, n, o), o)
            assert np.array_equal(bits, host(y) > 0)
            g = dy * bits
        gd = torch.from_numpy(g).cuda().double()
        xt = xd.double()
        if scheme != "exact":                    # the sample itself is tested elsewhere: x~ from the exported store
            ptr, col, val = B.rad_store_export_csr(ctx, st, n)
            xt = torch.zeros(n, d, dtype=torch.float64)
            rows = np.repeat(np.arange(n), np.diff(ptr))
            xt[torch.from_numpy(rows), torch.from_numpy(col.astype(np.int64))] = torch.from_numpy(val.astype(np.float64))
            xt = xt.cuda()
        B.rad_backward_dW(ctx, L, st, dyd, dW)
        assert_grad_close(host(dW), (xt.T @ gd).cpu().numpy(), TOL[B.RAD_BF16], n, "dW")
        B.rad_backward_dX(ctx, L, st, dyd, Wd, dX)
        assert_grad_close(host(dX), (gd @ Wd.double().T).cpu().numpy(), TOL[B.RAD_BF16], o, "dX", out_u=2 * U_BF16)
    finally:
        B.rad_store_destroy(st)


# (batch, d_in, d_out, scheme, fraction), the kernel of dX and that of dW whose loaders mask
@pytest.mark.parametrize("n,d,o,scheme,p,dX_kernel,dW_kernel", [
    (8200, 1001, 100, 1, 0.05, "dx_256", "dw_sparse_256x64"), (70, 33001, 200, 0, 1.0, "dx_256", "dw_dense_256"),
    (70, 33001, 255, 1, 0.05, "dx_256", "dw_sparse_256x256"), (1030, 400, 16201, 0, 1.0, "dx_128", "dw_dense_256"),
    (1030, 400, 16201, 1, 0.05, "dx_128", "dw_sparse_256x256"), (1030, 511, 16201, 1, 0.3, "dx_128", "dw_dense_256"),
    (2100, 500, 2050, 1, 0.02, "dx_128", "dw_sparse_splitk_256"), (2100, 500, 2050, 1, 0.08, "dx_128", "dw_sparse_splitk_256"),
    (12300, 300, 100, 0, 1.0, "dx_256x64", "dw_dense_128"), (90, 16300, 200, 0, 1.0, "dx_256x64", "dw_dense_256x64"),
    (1030, 500, 3001, 1, 0.05, "dx_128", "dw_sparse_256x64"), (1030, 500, 12301, 1, 0.08, "dx_128", "dw_sparse_256x128")])
def test_masks_in_the_loaders(ctx, n, d, o, scheme, p, dX_kernel, dW_kernel):
    """ReLU layers whose gradient is not masked ahead of the products: fewer than 256 outputs, or many rows of fewer than 512
    inputs.  dW and dX of the exported store and bits, and the kernels that form them."""
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import host, empty, unpack_bits, assert_grad_close, U_F32, U_BF16
    print("masks in the loaders", n, d, o, scheme, p, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(n + d + o)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16)  # noqa: E731
    x, W, dy = r(n, d), r(d, o), r(n, o)
    y, dW, dX = torch.empty_like(dy), empty((d, o)), torch.empty_like(x)
    layer = B.make_layer(n, d, o, dtype=B.RAD_BF16, relu=True)
    store = B.rad_store_create(ctx, layer, scheme, p)
    try:
        B.rad_forward_sample(ctx, layer, B.make_sampling(scheme, p, 5), x, W, None, y, store)
        B.rad_ctx_timing(ctx, None)
        B.rad_ctx_timing_reset(ctx)
        B.rad_backward_dW(ctx, layer, store, dy, dW)
        B.rad_backward_dX(ctx, layer, store, dy, W, dX)
        ran = {k: B.rad_ctx_timing_read(ctx, k)[0] for k in ("mask_rows", "dma", "gemm_bf16_" + dX_kernel, "gemm_bf16_" + dW_kernel,
                                                            "gemm_bf16_dx_256x64", "gemm_bf16_dw_dense_256x64")}
        bits = unpack_bits(B.rad_store_export_bits(ctx, store, n, o), o)
        csr = B.rad_store_export_csr(ctx, store, n) if scheme else None
    finally:
        B.rad_ctx_timing(ctx, "")
        B.rad_store_destroy(store)
    assert ran["mask_rows"] == ran["dma"] == 0
    assert ran["gemm_bf16_" + dX_kernel] == 1 and ran["gemm_bf16_" + dW_kernel] == 1
    assert ran["gemm_bf16_dx_256x64"] == (dX_kernel == "dx_256x64")                      # (their names hold the others')
    assert ran["gemm_bf16_dw_dense_256x64"] == (dW_kernel == "dw_dense_256x64")
    g = dy.double() * torch.from_numpy(bits).cuda()
    xt = x.double()
    if scheme:
        ptr, col, val = csr
        xt = torch.zeros(n, d, device="cuda", dtype=torch.float64)
        rows = np.repeat(np.arange(n), np.diff(ptr))
        xt[torch.from_numpy(rows).cuda(), torch.from_numpy(col.astype(np.int64)).cuda()] = torch.from_numpy(val.astype(np.float64)).cuda()
    assert_grad_close(host(dW), (xt.t().contiguous() @ g).cpu().numpy(), 1e-4, n, "dW", acc_u=U_F32)
    assert_grad_close(host(dX), (g @ W.double().t().contiguous()).cpu().numpy(), 2e-2, o, "dX", acc_u=U_F32, out_u=2 * U_BF16)
