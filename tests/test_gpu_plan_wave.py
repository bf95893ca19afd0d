"""The fixed-k draw of short rows (a wave per row) against the oracle's k smallest (key, column) pairs: widths around the
one, two and four Philox calls of a lane, rows that start inside a call, k from 1 to all columns, several steps' worth of
rows, and equal keys across the cut (keys shifted right)."""
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


WIDTHS = [1, 2, 3, 31, 100, 247, 248, 250, 255, 256, 257, 300, 504, 510, 512, 513, 784, 1015, 1016, 1018, 1024, 1025]


@pytest.mark.parametrize("cols", WIDTHS)
@pytest.mark.parametrize("p", [0.001, 0.1, 0.5, 0.97, 1.0])
def test_columns_of_every_row(ctx, cols, p):
    check_rows(ctx, cols, p, 0)


@pytest.mark.parametrize("cols", WIDTHS)
@pytest.mark.parametrize("p", [0.001, 0.1, 0.5, 0.97])
@pytest.mark.parametrize("shift", [22, 28, 31])
def test_equal_keys_across_the_cut(ctx, cols, p, shift):
    """Keys of 10, 4 and 1 bits: equal ones straddle the cut in most rows and go to the lowest columns."""
    check_rows(ctx, cols, p, shift)


def check_rows(ctx, cols, p, shift):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev
    rows, seed = 41, 12345678901234
    print("plan", cols, p, shift, flush=True)
    x = np.random.default_rng(cols).standard_normal((rows, cols)).astype(np.float32)
    L = B.make_layer(rows, cols, 8, relu=False)
    st = B.rad_store_create(ctx, L, B.RAD_FIXEDK_PER_EXAMPLE, p)
    B.rad_debug_key_shift(ctx, shift)
    try:
        B.rad_sample_pack(ctx, B.make_sampling(B.RAD_FIXEDK_PER_EXAMPLE, p, seed, 3, 5), dev(x), st)
        ptr, col, val = B.rad_store_export_csr(ctx, st, rows)
        k = R.fixed_k(p, cols)
        keys = R.element_keys(seed, 3, 5, 0, rows * cols).reshape(rows, cols) >> np.uint32(shift)
        order = np.lexsort((np.broadcast_to(np.arange(cols), keys.shape), keys), axis=1)[:, :k]
        want = np.sort(order, axis=1)
        assert np.array_equal(ptr, np.arange(rows + 1) * k)
        assert np.array_equal(col.reshape(rows, k), want)
        assert np.allclose(val.reshape(rows, k), np.take_along_axis(x, want, 1) * np.float32(cols / k), rtol=1e-6)
    finally:
        B.rad_debug_key_shift(ctx, 0)
        B.rad_store_destroy(st)
