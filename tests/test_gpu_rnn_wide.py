"""The recurrent model with a hidden state of 193 to 1024 units (a chunk of time steps per launch, W_hh in the registers of
the chip): widths around its 16- and 128-column ranges, batches around its groups and row tiles, lengths around its chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_rnn import ctx, run_rnn  # noqa: F401


def margin(d):
    """Smallest |pre-activation| over all examples, steps and units, in units of their root mean square."""
    x, h, low, sq, n = d["x"].astype(np.float64), 0.0, np.inf, 0.0, 0
    W_ih, W_hh, b = (d[k].astype(np.float64) for k in ("W_ih", "W_hh", "b"))
    for t in range(x.shape[1]):
        a = x[:, t] @ W_ih + b + (h @ W_hh if t else 0.0)
        low, sq, n, h = min(low, np.abs(a).min()), sq + np.square(a).sum(), n + a.size, np.maximum(a, 0.0)
    return low / np.sqrt(sq / n)


def data(seed, batch, T, hidden, d_input=1, classes=10, identity=False):
    """The first of the seeds from `seed` on whose pre-activations stay clear of zero: an fp32 sum of up to 1024 products
    is within about 3e-7 of their size (sqrt(1024) / 2 roundings of 6e-8 each at a third of it), and a ReLU bit that
    falls the other way for one example is no rounding error (128 x 600 units, 4 steps: one in three of the seeds)."""
    from paper_2007_10412_amd import synth
    for s in range(seed, seed + 1000):
        d = synth.rnn(seed=s, batch=batch, T=T, d_input=d_input, hidden=hidden, classes=classes, identity=identity)
        if margin(d) > 1e-6:
            return d
    raise AssertionError("no such data")


@pytest.mark.parametrize("hidden", [193, 256, 257, 383, 400, 512, 513, 528, 640, 700, 800, 896, 1000, 1023, 1024])
def test_widths(ctx, hidden):  # noqa: F811
    run_rnn(ctx, data(hidden, 20, 5, hidden), 1, 0.2, seed=3)


@pytest.mark.parametrize("batch", [1, 7, 8, 9, 127, 128, 129, 137, 185, 192, 193])
@pytest.mark.parametrize("hidden", [250, 600])
def test_batches(ctx, batch, hidden):  # noqa: F811
    run_rnn(ctx, data(batch, batch, 4, hidden), 3, 0.1, seed=4)


@pytest.mark.parametrize("T", [1, 2, 31, 32, 33, 34, 64, 65])
@pytest.mark.parametrize("scheme,p", [(0, 1.0), (1, 0.3), (2, 0.25), (4, 0.25), (5, 0.25)])
def test_lengths(ctx, T, scheme, p):  # noqa: F811
    run_rnn(ctx, data(T, 6, T, 210, d_input=3, classes=5), scheme, p, seed=T, check_store=T > 1)


@pytest.mark.parametrize("T,chunks", [(256, 8), (257, 8), (264, 8)])
@pytest.mark.parametrize("scheme,p", [(0, 1.0), (1, 0.3)])
def test_longer_chunks_of_longer_sequences(ctx, T, chunks, scheme, p):  # noqa: F811
    """An eighth of the sequence from 257 steps on (the last chunk shorter).  W_hh is the
    identity: with a random one the gradients of early steps leave the range of fp32."""
    from paper_2007_10412_amd import binding as B
    run_rnn(ctx, data(T, 2, T, 200, identity=True), scheme, p, seed=T)
    assert B.rad_debug_redone_launches(ctx) == (0, 2 * chunks)


def test_longest_chunks(ctx):  # noqa: F811
    """128 steps and one more chunk: nine launches per direction, and the bits of the stand-in."""
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty
    names, runs = ["W_ih", "W_hh", "b", "W_ho", "b_o"], []
    d = synth.rnn(seed=1, batch=9, T=1025, d_input=1, hidden=200, classes=10, identity=True)
    m = B.rad_model_create_rnn(ctx, 9, 1025, 1, 200, 10, 1, 0.3)
    try:
        params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
        for groups in (0, 0xff):
            B.rad_debug_absent_groups(ctx, groups, 18)
            B.rad_train_step(ctx, m, B.make_sampling(1, 0.3, 5, 20, 0), dev(d["x"]), dev(d["labels"]), params, grads)
            assert B.rad_debug_redone_launches(ctx) == (18 if groups else 0, 18)
            runs.append([host(g).copy() for g in grads])
        assert all(np.array_equal(a, b) and np.isfinite(a).all() for a, b in zip(*runs))
    finally:
        B.rad_model_destroy(m)


def test_transient_memory_of_long_chunks():
    """Chunks of 128 steps of 160 x 1000 (82 MB of dense h or g, the model's): what the step takes beside them is 32 MB of x~
    at most, four split sums of dW_hh (16 MB) and a few of flags and small sums, not another 82 MB of x~."""
    import torch
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, empty
    names, batch, T, hidden, took = ["W_ih", "W_hh", "b", "W_ho", "b_o"], 160, 1024, 1000, []
    d = synth.rnn(seed=1, batch=batch, T=T, d_input=1, hidden=hidden, classes=10, identity=True)
    params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
    x, labels = dev(d["x"]), dev(d["labels"])
    for _ in range(2):                       # the first one loads the kernels
        c = B.rad_ctx_create()
        m = B.rad_model_create_rnn(c, batch, T, 1, hidden, 10, 1, 0.05)
        try:
            torch.cuda.synchronize()
            before = torch.cuda.mem_get_info()[0]
            B.rad_train_step(c, m, B.make_sampling(1, 0.05, 5, 20, 0), x, labels, params, grads)
            torch.cuda.synchronize()
            took.append((before - torch.cuda.mem_get_info()[0]) / 1e6)
        finally:
            B.rad_model_destroy(m)
            B.rad_ctx_destroy(c)
    print("rnn wide transient MB", took, flush=True)
    assert took[1] < 72, took


@pytest.mark.parametrize("batch,hidden,T", [(128, 1024, 264), (160, 1000, 530)])
def test_parts_of_a_chunk_under_dW(ctx, batch, hidden, T):  # noqa: F811
    """Chunks of 33 steps (17 MB of x~, at once) and of 67 (43 MB, parts of 34 and 33): with every number kept, the gradients of
    the exact store, which takes a chunk at once, up to the order of the fp32 sums over steps x batch."""
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty, assert_grad_close, U_F32
    names, runs = ["W_ih", "W_hh", "b", "W_ho", "b_o"], []
    d = synth.rnn(seed=1, batch=batch, T=T, d_input=1, hidden=hidden, classes=10, identity=True)
    for scheme in (0, 1):
        m = B.rad_model_create_rnn(ctx, batch, T, 1, hidden, 10, scheme, 1.0)
        try:
            params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
            B.rad_train_step(ctx, m, B.make_sampling(scheme, 1.0, 5, 20, 0), dev(d["x"]), dev(d["labels"]), params, grads)
            runs.append([host(g).copy() for g in grads])
        finally:
            B.rad_model_destroy(m)
    for name, a, b in zip(names, *runs):
        assert_grad_close(b, a.astype(np.float64), 1e-4, T * batch, name, acc_u=U_F32, c=32.0)


@pytest.mark.parametrize("scheme,p", [(0, 1.0), (1, 0.1)])
@pytest.mark.parametrize("batch,hidden,T", [(100, 900, 34), (100, 1001, 34), (150, 770, 35)])
def test_split_rows_of_a_chunk(ctx, batch, hidden, T, scheme, p):  # noqa: F811
    """dW_hh of a chunk with its rows split (2048 rows and more at 1024 units), at widths that end inside a tile."""
    from paper_2007_10412_amd import binding as B
    B.rad_ctx_timing(ctx, "gemm_f32_dw_splitk_128")
    B.rad_ctx_timing_reset(ctx)
    try:
        run_rnn(ctx, data(batch, batch, T, hidden), scheme, p, seed=8)
        assert B.rad_ctx_timing_read(ctx, "gemm_f32_dw_splitk_128")[0] >= 1
    finally:
        B.rad_ctx_timing(ctx, "")


def test_wider_than_the_chip_holds(ctx):  # noqa: F811
    run_rnn(ctx, data(9, 6, 4, 1100), 1, 0.2, seed=5)


@pytest.mark.parametrize("hidden,batch", [(200, 20), (1024, 130)])
@pytest.mark.parametrize("scheme", [0, 1])
def test_chunks_whose_launch_gave_up(ctx, hidden, batch, scheme):  # noqa: F811
    """A wait bound of one look: some workgroup gives up at once, and the stand-in kernel computes the chunk."""
    from paper_2007_10412_amd import binding as B
    B.rad_debug_poll_limit(ctx, 1)
    run_rnn(ctx, data(hidden, batch, 40, hidden, d_input=2), scheme, 0.2 if scheme else 1.0, seed=6)
    redone, launches = B.rad_debug_redone_launches(ctx)
    assert launches == 4 and 1 <= redone <= 4


@pytest.mark.parametrize("hidden", [193, 250, 300, 511, 640, 690, 801, 1000, 1024])
@pytest.mark.parametrize("batch", [5, 150])
def test_the_stand_in_gives_the_same_bits(ctx, hidden, batch):  # noqa: F811
    """Loss, gradients and store of a step do not depend on which launches were computed again: none, the first, those of
    some examples only (whose groups are absent), all."""
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty
    T, names = 35, ["W_ih", "W_hh", "b", "W_ho", "b_o"]
    d = synth.rnn(seed=hidden, batch=batch, T=T, d_input=2, hidden=hidden, classes=10, identity=False)
    print("rnn wide bits", hidden, batch, flush=True)
    m = B.rad_model_create_rnn(ctx, batch, T, 2, hidden, 10, 1, 0.2)
    try:
        params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
        x, labels, runs = dev(d["x"]), dev(d["labels"]), []
        for groups, launches, redone in ((0, 0, 0), (0xff, 1, 1), (0x0a, 4, 4), (0xff, 4, 4)):
            for g in grads:
                g.fill_(float("nan"))
            B.rad_debug_absent_groups(ctx, groups, launches)
            loss = B.rad_train_step(ctx, m, B.make_sampling(1, 0.2, 5, 20, 0), x, labels, params, grads)
            assert B.rad_debug_redone_launches(ctx) == (redone, 4)
            runs.append([np.float32(loss)] + [host(g).copy() for g in grads] +
                        list(B.rad_store_export_csr(ctx, B.rad_model_store(m, 0), (T - 1) * batch)))
        for run in runs[1:]:
            assert all(np.array_equal(a, b) for a, b in zip(run, runs[0]))
        assert all(np.isfinite(a).all() for a in runs[0])
    finally:
        B.rad_model_destroy(m)


@pytest.mark.parametrize("T", [1, 2, 3, 33])
@pytest.mark.parametrize("groups", [0x01, 0x84, 0xff])
def test_groups_that_no_workgroup_reached(ctx, T, groups):  # noqa: F811
    """Nobody waits in a chunk of one time step, and nobody waits for a group without workgroups: what they left out shows
    in the groups' counters only.  Three groups of examples, the third of them with one example."""
    from paper_2007_10412_amd import binding as B
    launches = -(-T // 32) * (1 + (T > 1))
    for n in (1, launches):
        B.rad_debug_absent_groups(ctx, groups, n)
        run_rnn(ctx, data(T, 19, T, 250, d_input=2), 1, 0.3, seed=T, check_store=T > 1)
        assert B.rad_debug_redone_launches(ctx) == (n, launches)
    run_rnn(ctx, data(T, 19, T, 250, d_input=2), 1, 0.3, seed=T, check_store=T > 1)
    assert B.rad_debug_redone_launches(ctx) == (0, launches)


@pytest.mark.parametrize("failing,redone", [(1, 1), (2, 3), (4, 7), (14, 14)])
def test_failing_launches_are_not_repeated_at_once(ctx, failing, redone):  # noqa: F811
    """14 launches, the first ones of which find no workgroups: after the second failure in a row one launch goes to the
    stand-in without trying, then three, then seven."""
    from paper_2007_10412_amd import binding as B
    B.rad_debug_absent_groups(ctx, 0xff, failing)
    run_rnn(ctx, data(3, 6, 200, 200), 1, 0.2, seed=7)
    assert B.rad_debug_redone_launches(ctx) == (redone, 14)


@pytest.mark.parametrize("failing,redone", [(1, 1), (2, 2), (3, 4), (5, 7), (16, 16)])
def test_failing_launches_of_long_chunks(failing, redone):
    """16 launches of 98 steps, the first ones of which find no workgroups: what goes to the stand-in without trying counts in
    time steps (none after two failures in a row, one launch after three, two after four), and the numbers are those of an
    undisturbed step."""
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty
    names, runs, T = ["W_ih", "W_hh", "b", "W_ho", "b_o"], [], 784
    d = synth.rnn(seed=2, batch=6, T=T, d_input=1, hidden=200, classes=10, identity=True)
    c = B.rad_ctx_create()
    m = B.rad_model_create_rnn(c, 6, T, 1, 200, 10, 1, 0.2)
    try:
        params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
        for n, expected in ((0, 0), (failing, redone)):
            B.rad_debug_absent_groups(c, 0xff, n)
            B.rad_train_step(c, m, B.make_sampling(1, 0.2, 5, 20, 0), dev(d["x"]), dev(d["labels"]), params, grads)
            assert B.rad_debug_redone_launches(c) == (expected, 16)
            runs.append([host(g).copy() for g in grads])
        assert all(np.array_equal(a, b) and np.isfinite(a).all() for a, b in zip(*runs))
    finally:
        B.rad_model_destroy(m)
        B.rad_ctx_destroy(c)


@pytest.mark.parametrize("contexts,batch,hidden", [(2, 160, 600), (3, 128, 1000), (3, 20, 300)])
def test_models_of_several_contexts_at_once(contexts, batch, hidden):
    """Each on a stream of its own, steps enqueued in turn: the launches of one wait for, or give way to, those of another, and
    every step has the bits of a step taken alone."""
    import torch
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty
    T, names = 70, ["W_ih", "W_hh", "b", "W_ho", "b_o"]
    d = synth.rnn(seed=1, batch=batch, T=T, d_input=1, hidden=hidden, classes=10, identity=False)
    print("rnn wide contexts", contexts, batch, hidden, flush=True)
    sides = []
    try:
        for _ in range(contexts):
            stream = torch.cuda.Stream()
            c = B.rad_ctx_create(stream)
            sides.append((c, B.rad_model_create_rnn(c, batch, T, 1, hidden, 10, 1, 0.1), dev(d["x"]), dev(d["labels"]),
                          [dev(d[n]) for n in names], [empty(d[n].shape) for n in names], stream))
        torch.cuda.synchronize()

        def step(side, seed):
            B.rad_train_step(side[0], side[1], B.make_sampling(1, 0.1, seed, 20, 0), side[2], side[3], side[4], side[5],
                             want_loss=False)
        step(sides[0], 5)
        torch.cuda.synchronize()
        alone = [host(g).copy() for g in sides[0][5]]
        for _ in range(3):
            for seed in (1, 2, 5):
                for side in sides:
                    step(side, seed)
            torch.cuda.synchronize()
            print([B.rad_debug_redone_launches(side[0]) for side in sides], flush=True)
            for side in sides:
                assert all(np.array_equal(host(g), a) for g, a in zip(side[5], alone))
    finally:
        for side in sides:
            B.rad_model_destroy(side[1])
            B.rad_ctx_destroy(side[0])


@pytest.mark.parametrize("models", [[(128, 1000, 264), (128, 1000, 600), (128, 1000, 264)], [(192, 1000, 300), (160, 900, 420)]])
def test_long_chunks_of_several_contexts_at_once(models):
    """Chunks of 33 to 75 steps of models of different lengths, each on a stream of its own: every step has the bits of one
    taken alone."""
    import torch
    from paper_2007_10412_amd import binding as B, synth
    from tests.gpu_util import dev, host, empty
    names, sides, alone = ["W_ih", "W_hh", "b", "W_ho", "b_o"], [], []
    try:
        for k, (batch, hidden, T) in enumerate(models):
            d = synth.rnn(seed=k, batch=batch, T=T, d_input=1, hidden=hidden, classes=10, identity=True)
            print("rnn wide contexts", batch, hidden, T, flush=True)
            c = B.rad_ctx_create(torch.cuda.Stream())
            sides.append((c, B.rad_model_create_rnn(c, batch, T, 1, hidden, 10, 1, 0.1), dev(d["x"]), dev(d["labels"]),
                          [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]))
        torch.cuda.synchronize()

        def step(side):
            B.rad_train_step(side[0], side[1], B.make_sampling(1, 0.1, 5, 20, 0), side[2], side[3], side[4], side[5], want_loss=False)
        for side in sides:
            step(side)
            torch.cuda.synchronize()
            alone.append([host(g).copy() for g in side[5]])
        for _ in range(4):
            for side in sides:
                step(side)
        torch.cuda.synchronize()
        print([B.rad_debug_redone_launches(side[0]) for side in sides], flush=True)
        for side, want in zip(sides, alone):
            assert all(np.array_equal(host(g), a) and np.isfinite(a).all() for g, a in zip(side[5], want))
    finally:
        for side in sides:
            B.rad_model_destroy(side[1])
            B.rad_ctx_destroy(side[0])


def test_stream_kept_to_a_part_of_the_chip():
    """The workgroups of a chunk's launch could not all run on such a stream: its models take a launch per time step."""
    import ctypes
    import torch
    from paper_2007_10412_amd import binding as B
    torch.zeros(1, device="cuda")
    hip = ctypes.CDLL("libamdhip64.so")
    stream, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*([0x0fffffff] * 8))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    c = B.rad_ctx_create(torch.cuda.ExternalStream(stream.value))
    try:
        run_rnn(c, data(2, 9, 40, 300), 1, 0.2, seed=6)
        assert B.rad_debug_redone_launches(c) == (0, 0)
    finally:
        B.rad_ctx_destroy(c)
        assert hip.hipStreamDestroy(stream) == 0


def test_repeated_steps_are_identical(ctx):  # noqa: F811
    from paper_2007_10412_amd import binding as B
    from tests.gpu_util import dev, host, empty
    d = data(11, 70, 70, 360)
    names = ["W_ih", "W_hh", "b", "W_ho", "b_o"]
    m = B.rad_model_create_rnn(ctx, 70, 70, 1, 360, 10, 1, 0.1)
    try:
        params, grads = [dev(d[n]) for n in names], [empty(d[n].shape) for n in names]
        x, labels, runs = dev(d["x"]), dev(d["labels"]), []
        for _ in range(3):
            B.rad_train_step(ctx, m, B.make_sampling(1, 0.1, 5, 20, 0), x, labels, params, grads)
            runs.append([host(g).copy() for g in grads])
        assert all(np.array_equal(a, b) for r in runs[1:] for a, b in zip(r, runs[0]))
    finally:
        B.rad_model_destroy(m)
