"""dW of a bf16 layer whose store has more entries in a row's bucket of 256 columns than the kernel holds in registers (24 or
56): keys of one bit, drawn with the test hook, put all of a row's entries into its lowest columns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2007_10412_amd import binding as B
    c = B.rad_ctx_create()
    yield c
    B.rad_ctx_destroy(c)


@pytest.mark.parametrize("batch,d_in,d_out", [(40, 1024, 72), (300, 1000, 130), (2100, 1024, 200), (2300, 2300, 2300), (2048, 2816, 3080)])
@pytest.mark.parametrize("p", [0.03, 0.1])
@pytest.mark.parametrize("relu,beta", [(False, 0), (True, 0), (False, 1)])
def test_dW(ctx, batch, d_in, d_out, p, relu, beta):
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import host, assert_grad_close, U_F32
    print("dW long segments", batch, d_in, d_out, p, relu, beta, flush=True)
    rng = torch.Generator(device="cuda").manual_seed(batch + d_in + d_out)
    r = lambda *shape: torch.randn(*shape, device="cuda", generator=rng).to(torch.bfloat16)  # noqa: E731
    x, W, dy = r(batch, d_in), r(d_in, d_out), r(batch, d_out)
    y, dW = torch.empty_like(dy), torch.ones(d_in, d_out, device="cuda")
    layer = B.make_layer(batch, d_in, d_out, dtype=B.RAD_BF16, relu=relu)
    store = B.rad_store_create(ctx, layer, B.RAD_FIXEDK_PER_EXAMPLE, p)
    try:
        B.rad_debug_key_shift(ctx, 31)
        B.rad_forward_sample(ctx, layer, B.make_sampling(B.RAD_FIXEDK_PER_EXAMPLE, p, 7, 0, 0), x, W, None, y, store)
        B.rad_backward_dW(ctx, layer, store, dy, dW, beta=float(beta))
        rp, col, val = B.rad_store_export_csr(ctx, store, batch)
    finally:
        B.rad_store_destroy(store)
    rows = np.repeat(np.arange(batch), np.diff(rp))
    longest = np.bincount(rows * ((d_in + 255) // 256) + col // 256).max()
    assert longest > (24 if p == 0.03 else 56), longest
    xs = torch.zeros(batch, d_in, device="cuda", dtype=torch.float64)
    xs[torch.from_numpy(rows).cuda(), torch.from_numpy(col.astype(np.int64)).cuda()] = torch.from_numpy(val.astype(np.float64)).cuda()
    g = dy.double() * (y > 0) if relu else dy.double()
    want = (xs.t().contiguous() @ g).cpu().numpy() + beta
    assert_grad_close(host(dW), want, 1e-4, batch, "dW", acc_u=U_F32)


def test_one_long_segment_costs_little(ctx):
    """65536 x 1000 at fraction 0.0294: one of the two Bernoulli draws has a segment of 25 entries, one more than the kernel
    holds, the other has none.  dW of both against the product of the exported store, and its time with the long segment
    below one and a half times that without (all rows are looked over for it: 4.6 times with a wave to a row)."""
    import torch
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import host, assert_grad_close, U_F32
    batch, d_in, d_out, p = 65536, 1000, 64, 0.0294
    print("dW with one long segment", flush=True)
    rng = torch.Generator(device="cuda").manual_seed(5)
    x, dy = (torch.randn(batch, n, device="cuda", generator=rng).to(torch.bfloat16) for n in (d_in, d_out))
    dW, layer = torch.empty(d_in, d_out, device="cuda"), B.make_layer(batch, d_in, d_out, dtype=B.RAD_BF16, relu=False)
    store, us = B.rad_store_create(ctx, layer, B.RAD_BERNOULLI, p), {}
    try:
        for seed, longest in ((1, 22), (25, 25)):
            B.rad_sample_pack(ctx, B.make_sampling(B.RAD_BERNOULLI, p, seed, 0, 0), x, store)
            rp, col, val = B.rad_store_export_csr(ctx, store, batch)
            rows = np.repeat(np.arange(batch), np.diff(rp))
            assert np.bincount(rows * 4 + col // 256).max() == longest
            times = []
            for _ in range(9):
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                torch.cuda.synchronize()
                ev[0].record()
                B.rad_backward_dW(ctx, layer, store, dy, dW)
                ev[1].record()
                torch.cuda.synchronize()
                times.append(1e3 * ev[0].elapsed_time(ev[1]))
            us[longest] = np.median(times)
            xs = torch.zeros(batch, d_in, device="cuda", dtype=torch.float64)
            xs[torch.from_numpy(rows).cuda(), torch.from_numpy(col.astype(np.int64)).cuda()] = torch.from_numpy(val.astype(np.float64)).cuda()
            assert_grad_close(host(dW), (xs.t().contiguous() @ dy.double()).cpu().numpy(), 1e-4, batch, "dW", acc_u=U_F32)
    finally:
        B.rad_store_destroy(store)
    print(us, flush=True)
    assert us[25] < 1.5 * us[22], us
