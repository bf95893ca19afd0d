"""GPU parity of the fp32 forward and dX products of small layers (16 x 32 tiles, K split over the waves of a workgroup)
against fp64: shapes around the tiles, the 64-deep passes and the waves' shares, on both sides of the rule that chooses
this kernel, with ReLU bits on either side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2007_10412_amd import binding as B
    c = B.rad_ctx_create()
    yield c
    B.rad_ctx_destroy(c)


@pytest.mark.parametrize("n,d,o", [(1, 64, 1), (3, 65, 112), (15, 113, 31), (16, 63, 33), (17, 129, 113), (150, 784, 300),
                                   (33, 511, 200), (300, 520, 700), (40, 2047, 10), (40, 2049, 10), (512, 200, 1000),
                                   (513, 1023, 130), (700, 128, 520), (64, 513, 512)])
@pytest.mark.parametrize("relu", [False, True])
def test_layer(ctx, n, d, o, relu):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty, unpack_bits, assert_grad_close, TOL
    rng = np.random.default_rng(n + 7 * d + 13 * o)
    x = rng.standard_normal((n, d)).astype(np.float32)
    W = (rng.standard_normal((d, o)) / np.sqrt(d)).astype(np.float32)
    b = rng.standard_normal(o).astype(np.float32)
    dy = rng.standard_normal((n, o)).astype(np.float32)
    print("layer", n, d, o, relu, flush=True)
    L = B.make_layer(n, d, o, relu=relu, has_bias=True)
    st = B.rad_store_create(ctx, L, B.RAD_FIXEDK_PER_EXAMPLE, 0.2)
    try:
        y, dX = empty((n, o)), empty((n, d))
        Wd = dev(W)
        B.rad_forward_sample(ctx, L, B.make_sampling(B.RAD_FIXEDK_PER_EXAMPLE, 0.2, 5), dev(x), Wd, dev(b), y, st)
        h = x.astype(np.float64) @ W.astype(np.float64) + b
        assert_grad_close(host(y), np.maximum(h, 0) if relu else h, TOL[B.RAD_F32], d, "y")
        g = dy.astype(np.float64)
        if relu:
            bits = unpack_bits(B.rad_store_export_bits(ctx, st, n, o), o)
            assert np.array_equal(bits, host(y) > 0)
            g = g * bits
        B.rad_backward_dX(ctx, L, st, dev(dy), Wd, dX)
        assert_grad_close(host(dX), g @ W.astype(np.float64).T, TOL[B.RAD_F32], o, "dX")
    finally:
        B.rad_store_destroy(st)


@pytest.mark.parametrize("n,k,o,fwd,dx", [(16, 2048, 32, True, True), (16, 2048, 512, True, True), (32, 3072, 64, False, True), (32, 3072, 128, True, True),
                                          (32, 4096, 64, False, True), (16, 8192, 64, False, True), (16, 4096, 2048, True, True),
                                          (32, 4096, 4096, True, True), (48, 4096, 4096, False, False), (64, 2048, 4096, True, True)])
def test_long_contractions_of_whole_tiles(ctx, n, k, o, fwd, dx):
    """Forward n x k x o and dX of the same output and contraction: the route that was measured as the faster one, and the
    product."""
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty, assert_grad_close, TOL
    rng = np.random.default_rng(n + k + o)
    a, w = rng.standard_normal((n, k)).astype(np.float32), (rng.standard_normal((k, o)) / np.sqrt(k)).astype(np.float32)
    want = a.astype(np.float64) @ w.astype(np.float64)
    print("whole tiles", n, k, o, flush=True)
    for forward, here in ((True, fwd), (False, dx)):
        L = B.make_layer(n, k, o, relu=False) if forward else B.make_layer(n, o, k, relu=False)
        st = B.rad_store_create(ctx, L, B.RAD_EXACT, 1.0)
        B.rad_ctx_timing(ctx, "gemm_f32_%s_ks" % ("fwd" if forward else "dx"))
        B.rad_ctx_timing_reset(ctx)
        try:
            out = empty((n, o))
            if forward:
                B.rad_forward_sample(ctx, L, B.make_sampling(B.RAD_EXACT, 1.0, 5), dev(a), dev(w), None, out, st)
            else:
                B.rad_backward_dX(ctx, L, st, dev(a), dev(np.ascontiguousarray(w.T)), out)
            assert_grad_close(host(out), want, TOL[B.RAD_F32], k, "forward" if forward else "dX")
            assert (B.rad_ctx_timing_read(ctx, None)[0] == 1) == here
        finally:
            B.rad_ctx_timing(ctx, "")
            B.rad_ctx_timing_reset(ctx)
            B.rad_store_destroy(st)
