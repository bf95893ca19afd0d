"""GPU parity of the bf16 GEMMs whose rows start at any element: widths and batches that are multiples of nothing, so
that 16-byte loads and stores are aligned to an element only, chunks run past the end of a row and the last slices are
guarded.  The three calls of one layer (ReLU bits as loader masks) and a layer without ReLU, against the oracle, at
contraction lengths that end the pipeline at every point."""
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
