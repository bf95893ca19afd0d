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
