"""GPU parity of the bias gradient (column sums under the ReLU bits) at the rows and widths where its launch changes form
(one range of rows or several, a column or a 16-byte vector per lane, ragged last vectors), and of the backward calls of
wide bf16 layers whose masked gradient is written out for the direct-to-LDS GEMMs."""
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


def backward(ctx, n, d, o, dt, relu, sch, p, beta):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty, pack_bits
    import torch
    rng = np.random.default_rng(n + 3 * o + relu)
    rnd = R.round_bf16 if dt == B.RAD_BF16 else (lambda a: a)
    x = rnd(rng.standard_normal((n, d)).astype(np.float32))
    W = rnd((rng.standard_normal((d, o)) / np.sqrt(o)).astype(np.float32))
    dy = rnd(rng.standard_normal((n, o)).astype(np.float32))
    L = B.make_layer(n, d, o, dtype=dt, relu=relu, has_bias=True)
    st = B.rad_store_create(ctx, L, sch, p)
    try:
        B.rad_sample_pack(ctx, B.make_sampling(sch, p, 3), dev(x, dt), st)
        g = dy
        if relu:
            on = rng.random((n, o)) < 0.5
            B.rad_store_import_bits(ctx, st, pack_bits(on))
            g = dy * on
        dW, db, dX = empty((d, o)), empty((o,)), empty((n, d), dt)
        dW.zero_(); db.fill_(1.0)
        B.rad_backward_dW(ctx, L, st, dev(dy, dt), dW, db, beta)
        B.rad_backward_dX(ctx, L, st, dev(dy, dt), dev(W, dt), dX)
        xt = np.zeros((n, d), dtype=np.float32)
        if sch == B.RAD_EXACT:
            xt = x
        else:
            ptr, col, val = B.rad_store_export_csr(ctx, st, n)
            xt[np.repeat(np.arange(n), np.diff(ptr)), col] = val
        gd = torch.from_numpy(g).cuda().double()
        want = {"db": g.astype(np.float64).sum(0) + (1.0 if beta else 0.0),
                "dW": (torch.from_numpy(xt).cuda().double().T @ gd).cpu().numpy(),
                "dX": (gd @ torch.from_numpy(W).cuda().double().T).cpu().numpy()}
        return {"db": host(db), "dW": host(dW), "dX": host(dX)}, want
    finally:
        B.rad_store_destroy(st)


@pytest.mark.parametrize("n", [1, 15, 65, 512, 513, 1000])
@pytest.mark.parametrize("o", [1, 64, 70, 511, 512, 519])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("relu,beta", [(False, 0.0), (True, 1.0)])
def test_bias_gradient(ctx, n, o, dtype, relu, beta):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import assert_grad_close, TOL
    print("bias gradient", n, o, dtype, relu, flush=True)
    dt = B.RAD_BF16 if dtype == "bf16" else B.RAD_F32
    got, want = backward(ctx, n, 40, o, dt, relu, B.RAD_FIXEDK_PER_EXAMPLE, 0.2, beta)
    assert_grad_close(got["db"], want["db"], TOL[B.RAD_F32], n, "db")


@pytest.mark.parametrize("n,d,o", [(2048, 4096, 520), (4096, 4096, 2048), (4096, 2048, 4096)])
@pytest.mark.parametrize("scheme", ["exact", "per_example"])
def test_wide_layer_with_relu(ctx, n, d, o, scheme):
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import assert_grad_close, TOL, U_BF16
    print("wide layer", n, d, o, scheme, flush=True)
    sch, p = (B.RAD_EXACT, 1.0) if scheme == "exact" else (B.RAD_FIXEDK_PER_EXAMPLE, 0.1)
    got, want = backward(ctx, n, d, o, B.RAD_BF16, True, sch, p, 0.0)
    assert_grad_close(got["db"], want["db"], TOL[B.RAD_F32], n, "db")
    assert_grad_close(got["dW"], want["dW"], TOL[B.RAD_BF16], n, "dW")
    assert_grad_close(got["dX"], want["dX"], TOL[B.RAD_BF16], o, "dX", out_u=2 * U_BF16)
