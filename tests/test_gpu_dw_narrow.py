"""GPU parity of the dW of narrow layers from a compressed store against the oracle's product with the exported sample, on
both sides of the rule that chooses the row-split kernel: widths around its vectors and parts, rows around its groups of 8
and 32, columns around a 256-column bucket, ReLU bits, accumulation, one split, and rows with more entries than it holds
in registers."""
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


@pytest.mark.parametrize("n,d", [(1, 3), (7, 255), (31, 256), (33, 257), (150, 784), (2500, 1000)])
@pytest.mark.parametrize("o", [1, 4, 10, 12, 13, 16, 17, 33, 100, 128])
@pytest.mark.parametrize("dtype,scheme,p", [("f32", "bernoulli", 0.1), ("f32", "per_example", 0.7),
                                            ("bf16", "per_example", 0.1), ("bf16", "bernoulli", 0.15),
                                            ("f32", "replace_shared", 0.3)])
def test_narrow_dW(ctx, n, d, o, dtype, scheme, p):
    check_dW(ctx, n, d, o, dtype, scheme, p)


def check_here(ctx, *case):
    """check_dW, with both of its calls on the row-split kernel."""
    from paper_2007_10412_amd import binding as B
    B.rad_ctx_timing(ctx, "dw_narrow")
    B.rad_ctx_timing_reset(ctx)
    try:
        check_dW(ctx, *case)
        assert B.rad_ctx_timing_read(ctx, None)[0] == 2
    finally:
        B.rad_ctx_timing(ctx, "")
        B.rad_ctx_timing_reset(ctx)


@pytest.mark.parametrize("n", [65, 71, 72, 73, 95, 96, 97])
@pytest.mark.parametrize("d", [3, 255, 256, 257])
@pytest.mark.parametrize("o", [1, 4, 5, 12])
@pytest.mark.parametrize("dtype,scheme,p", [("f32", "bernoulli", 0.1), ("f32", "per_example", 0.7), ("bf16", "per_example", 0.1),
                                            ("bf16", "bernoulli", 0.5), ("bf16", "replace_shared", 0.3)])
def test_edges_of_groups_and_buckets(ctx, n, d, o, dtype, scheme, p):
    check_here(ctx, n, d, o, dtype, scheme, p)


@pytest.mark.parametrize("n,d", [(257, 255), (300, 513), (320, 256)])
@pytest.mark.parametrize("o", [13, 16, 17, 33, 100, 128, 129])
@pytest.mark.parametrize("scheme,p", [("bernoulli", 0.1), ("per_example", 0.7)])
def test_widths_of_several_parts(ctx, n, d, o, scheme, p):
    check_here(ctx, n, d, o, "f32", scheme, p)


def test_one_split(ctx):
    """256 buckets by three parts: the rows are not split and the kernel writes (and accumulates into) dW itself."""
    check_here(ctx, 300, 65535, 40, "f32", "bernoulli", 0.02)
    check_here(ctx, 300, 65535, 41, "f32", "bernoulli", 0.3)


@pytest.mark.parametrize("n,d,o", [(512, 300, 300), (700, 1030, 515), (160, 257, 290)])
def test_wider_fp32_layers(ctx, n, d, o):
    check_dW(ctx, n, d, o, "f32", "per_example", 0.1)


def check_dW(ctx, n, d, o, dtype, scheme, p):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty, unpack_bits, assert_grad_close, pack_bits, TOL
    dt = B.RAD_BF16 if dtype == "bf16" else B.RAD_F32
    sch = {"bernoulli": B.RAD_BERNOULLI, "per_example": B.RAD_FIXEDK_PER_EXAMPLE,
           "replace_shared": B.RAD_REPLACE_SHARED}[scheme]
    rng = np.random.default_rng(n + 7 * d + 13 * o)
    rnd = R.round_bf16 if dt == B.RAD_BF16 else (lambda a: a)
    x = rnd(rng.standard_normal((n, d)).astype(np.float32))
    dy = rnd(rng.standard_normal((n, o)).astype(np.float32))
    relu = (n + o) % 2 == 1
    print("narrow dW", n, d, o, dtype, scheme, flush=True)
    L = B.make_layer(n, d, o, dtype=dt, relu=relu)
    st = B.rad_store_create(ctx, L, sch, p)
    try:
        B.rad_sample_pack(ctx, B.make_sampling(sch, p, 3), dev(x, dt), st)
        ptr, col, val = B.rad_store_export_csr(ctx, st, n)
        xt = np.zeros((n, d))
        xt[np.repeat(np.arange(n), np.diff(ptr)), col] = val
        g = dy
        if relu:
            on = rng.random((n, o)) < 0.5
            B.rad_store_import_bits(ctx, st, pack_bits(on))
            g = dy * on
        want = xt.T @ g.astype(np.float64)
        dW = empty((d, o))
        B.rad_backward_dW(ctx, L, st, dev(dy, dt), dW)
        assert_grad_close(host(dW), want, TOL[B.RAD_F32], n, "dW")
        B.rad_backward_dW(ctx, L, st, dev(dy, dt), dW, beta=1.0)
        assert_grad_close(host(dW), 2 * want, TOL[B.RAD_F32], n, "dW + dW")
    finally:
        B.rad_store_destroy(st)


@pytest.mark.parametrize("n,d,o,p,here", [(150, 784, 10, 0.1, True), (65, 4096, 128, 0.1, False), (200, 4096, 128, 0.1, False),
                                          (600, 4096, 128, 0.1, True), (200, 784, 300, 0.1, False), (200, 784, 300, 0.5, True),
                                          (512, 1024, 1024, 0.1, False), (512, 1024, 1024, 0.5, True), (64, 784, 10, 0.1, False)])
def test_faster_route(ctx, n, d, o, p, here):
    """The side that was measured as the faster one is taken, and the product is right on both."""
    from paper_2007_10412_amd import binding as B
    if here:
        return check_here(ctx, n, d, o, "f32", "per_example", p)
    B.rad_ctx_timing(ctx, "dw_narrow")
    B.rad_ctx_timing_reset(ctx)
    try:
        check_dW(ctx, n, d, o, "f32", "per_example", p)
        assert B.rad_ctx_timing_read(ctx, None)[0] == 0
    finally:
        B.rad_ctx_timing(ctx, "")
        B.rad_ctx_timing_reset(ctx)


def check_small(ctx, *case):
    """check_dW, with both of its calls on the one-pass kernel for few rows."""
    from paper_2007_10412_amd import binding as B
    B.rad_ctx_timing(ctx, "dw_small")
    B.rad_ctx_timing_reset(ctx)
    try:
        check_dW(ctx, *case)
        assert B.rad_ctx_timing_read(ctx, None)[0] == 2
    finally:
        B.rad_ctx_timing(ctx, "")
        B.rad_ctx_timing_reset(ctx)


@pytest.mark.parametrize("n", [97, 127, 128, 129, 241, 255, 256])               # rows of eight waves, even a wave, the most
@pytest.mark.parametrize("d,o", [(31, 13), (32, 32), (33, 33), (257, 65), (784, 300), (300, 31)])
@pytest.mark.parametrize("scheme,p", [("bernoulli", 0.1), ("per_example", 0.02), ("replace_shared", 0.2)])
def test_few_rows(ctx, n, d, o, scheme, p):
    """Up to 256 fp32 rows on 32 x 32 tiles; three near-ties of 51 and 60 entries a row are the row split's."""
    split = (n, d, o) in [(128, 257, 65), (128, 300, 31), (256, 300, 31)] and p == 0.2
    (check_here if split else check_small)(ctx, n, d, o, "f32", scheme, p)


@pytest.mark.parametrize("n,d,o,p", [(49, 300, 64, 0.02), (56, 784, 300, 0.02), (64, 784, 300, 0.1), (65, 784, 301, 0.1), (80, 300, 65, 0.1),
                                     (96, 2000, 31, 0.05)])
def test_fewer_rows(ctx, n, d, o, p):
    """Waves with a few rows, the last ones with none."""
    check_small(ctx, n, d, o, "f32", "bernoulli", p)


def test_few_rows_long_segments(ctx):
    """Rows with more entries in a bucket than the kernel holds in registers."""
    check_small(ctx, 100, 784, 300, "f32", "bernoulli", 0.4)


@pytest.mark.parametrize("n,d,o,p", [(100, 784, 301, 0.4), (101, 784, 300, 0.4)])
def test_few_masked_rows_long_segments(ctx, n, d, o, p):
    """The same under ReLU bits, written and accumulated."""
    check_small(ctx, n, d, o, "f32", "bernoulli", p)
