"""The work that users of this library have it do, as cases that a timer can prepare and run.

Every path goes through the public entry points of `paper_2007_10412_amd.binding`, at the sizes of this repository's
configurations, tests and benchmark, and at generic sizes between and around them.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program has in hand before the call, on the GPU
    run(state)          one pass; returns its outputs
    work(case)          bytes and operations one pass cannot do without
    tolerance(case)     how far two correct implementations may be apart
"""
import math
import weakref

import torch

from paper_2007_10412_amd import binding as B

SCHEMES = {"exact": B.RAD_EXACT, "bernoulli": B.RAD_BERNOULLI, "shared": B.RAD_FIXEDK_SHARED,
           "per_example": B.RAD_FIXEDK_PER_EXAMPLE, "replace_per_example": B.RAD_REPLACE_PER_EXAMPLE,
           "project": B.RAD_PROJECT_SHARED}
PDE_D, PDE_DT = 0.25, 1.0 / 4096


def listed():
    return [
        # The smallest unit of use: the three calls of one fp32 layer (forward + sample, dW, dX) on a minibatch of 150
        # MNIST-sized inputs.  Latency and launches are all there is.
        {"name": "layer_784x300_f32", "path": "layer", "dtype": "f32", "batch": 150, "d_in": 784, "d_out": 300,
         "relu": True, "bias": False, "scheme": "bernoulli", "p": 0.1},
        # The same three calls where a wide bf16 layer of somebody's own model is trained with them.
        {"name": "layer_4096_bf16", "path": "layer", "dtype": "bf16", "batch": 4096, "d_in": 4096, "d_out": 4096,
         "relu": True, "bias": True, "scheme": "per_example", "p": 0.1},
        # Whole training step of the small MNIST network, fp32 with biases.
        {"name": "mlp_784_f32", "path": "mlp", "dtype": "f32", "batch": 150, "dims": "784-300-300-10", "bias": True,
         "scheme": "per_example", "p": 0.1, "index_free": False},
        # The benchmark's default: the wide bf16 network, a different sample for every example.
        {"name": "mlp_4096_bf16_per_example", "path": "mlp", "dtype": "bf16", "batch": 4096,
         "dims": "4096-4096-4096-1000", "bias": False, "scheme": "per_example", "p": 0.1, "index_free": False},
        # The same network with one sample for the whole minibatch.
        {"name": "mlp_4096_bf16_shared", "path": "mlp", "dtype": "bf16", "batch": 4096,
         "dims": "4096-4096-4096-1000", "bias": False, "scheme": "shared", "p": 0.1, "index_free": False},
        # A medium network whose sizes are multiples of nothing: batch, widths and class count as they come.
        {"name": "mlp_ragged_bf16", "path": "mlp", "dtype": "bf16", "batch": 1000, "dims": "1100-2050-1530-100",
         "bias": True, "scheme": "bernoulli", "p": 0.1, "index_free": False},
        # Training step of the small CIFAR-10 network (3 convolutions, 2 max pools, a linear layer).
        {"name": "cnn_32x32_f32", "path": "cnn", "batch": 150, "channels": "3-16-32-64", "pool": "0-1-1", "ksize": 3,
         "hw": 32, "classes": 10, "scheme": "bernoulli", "p": 0.1},
        # Back-propagation through time over 784 steps, hidden 1024: the longest training step.
        {"name": "rnn_1024_f32", "path": "rnn", "batch": 128, "T": 784, "hidden": 1024, "classes": 10,
         "scheme": "bernoulli", "p": 0.1},
        # The paper's own recurrent network (hidden 100, batch 150): a chain of very small steps.
        {"name": "rnn_100_f32", "path": "rnn", "batch": 150, "T": 784, "hidden": 100, "classes": 10,
         "scheme": "per_example", "p": 0.1},
        # Activation compression by itself on a 1 GiB stream: somebody's own forward pass, whose 4096-wide input to the
        # 10 class scores is sampled here and whose weight gradient is formed from the store.
        {"name": "sample_65536x4096_f32", "path": "sample", "dtype": "f32", "rows": 65536, "cols": 4096, "d_out": 10,
         "scheme": "bernoulli", "p": 0.1},
        # Adam over the parameters of the wide bf16 network (fp32 master copies).
        {"name": "adam_4096_bf16", "path": "optimizer", "kind": "adam", "dtype": "bf16",
         "counts": "16777216-16777216-4096000"},
        # The reaction-diffusion study at the paper's size, a control vector per compute unit.
        {"name": "pde_32x40960", "path": "pde", "n": 32, "steps": 40960, "problems": 256, "p": 0.01},
    ]


# ------------------------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: as it comes, or a whole multiple of 8 or 64 as widths are often chosen."""
    w = _log(rng, lo, hi)
    m = rng.choice((1, 1, 8, 64))
    return max(m, w // m * m)


def _fraction(rng):
    return rng.choice((0.5, 0.1, 0.1, 0.05, 0.02, round(rng.uniform(0.02, 0.5), 3)))


def _draw_layer(rng):
    bf16 = rng.random() < 0.5
    scheme = rng.choice(("bernoulli", "shared", "per_example", "per_example", "replace_per_example"))
    return {"path": "layer", "dtype": "bf16" if bf16 else "f32",
            "batch": _log(rng, 128, 8192) if bf16 else _log(rng, 16, 1024),
            "d_in": _width(rng, 256, 6144) if bf16 else _width(rng, 64, 2048),
            "d_out": _width(rng, 128, 6144) if bf16 else _width(rng, 10, 1024),
            "relu": rng.random() < 0.75, "bias": rng.random() < 0.5, "scheme": scheme, "p": _fraction(rng)}


def _draw_mlp(rng):
    bf16 = rng.random() < 0.6
    depth = rng.randint(1, 4)
    if bf16:
        batch = _log(rng, 128, 8192)
        dims = [_width(rng, 256, 4096) for _ in range(depth)] + [rng.choice((10, 100, 1000, _log(rng, 10, 2048)))]
    else:
        batch = _log(rng, 16, 512)
        dims = [_width(rng, 64, 1024) for _ in range(depth)] + [rng.choice((10, _log(rng, 2, 100)))]
    scheme = rng.choice(("per_example", "per_example", "shared", "bernoulli", "exact", "replace_per_example", "project"))
    return {"path": "mlp", "dtype": "bf16" if bf16 else "f32", "batch": batch, "dims": "-".join(map(str, dims)),
            "bias": rng.random() < 0.5, "scheme": scheme, "p": 1.0 if scheme == "exact" else _fraction(rng),
            "index_free": scheme in ("per_example", "bernoulli") and rng.random() < 0.25}


def _draw_cnn(rng):
    hw = rng.choice((16, 32))
    n = rng.randint(1, 4)
    channels = [rng.choice((1, 3))] + [rng.choice((8, 12, 16, 24, 32, 48, 64)) for _ in range(n)]
    pool, size, kind = [], hw, rng.choice((1, 2))
    for _ in range(n):
        p = kind if size >= 16 and rng.random() < 0.5 else 0
        size = size // 2 if p else size
        pool.append(p)
    return {"path": "cnn", "batch": _log(rng, 16, 512), "channels": "-".join(map(str, channels)),
            "pool": "-".join(map(str, pool)), "ksize": rng.choice((3, 3, 5)), "hw": hw, "classes": 10,
            "scheme": rng.choice(("bernoulli", "per_example")), "p": _fraction(rng)}


def _draw_rnn(rng):
    return {"path": "rnn", "batch": _log(rng, 16, 192), "T": _log(rng, 49, 784), "hidden": _width(rng, 64, 1024),
            "classes": 10, "scheme": rng.choice(("bernoulli", "per_example", "shared")), "p": _fraction(rng)}


def _draw_sample(rng):
    rows, cols = _log(rng, 1024, 65536), _width(rng, 256, 4096)
    return {"path": "sample", "dtype": rng.choice(("f32", "bf16")), "rows": rows, "cols": cols,
            "d_out": rng.choice((10, 10, 16, 100)), "scheme": rng.choice(("bernoulli", "per_example")), "p": _fraction(rng)}


def _draw_optimizer(rng):
    counts = [_log(rng, 10, 16777216) for _ in range(rng.randint(1, 8))]
    return {"path": "optimizer", "kind": rng.choice(("adam", "sgd")), "dtype": rng.choice(("f32", "bf16")),
            "counts": "-".join(map(str, counts))}


def _draw_pde(rng):
    return {"path": "pde", "n": rng.randint(8, 32), "steps": _log(rng, 1024, 40960), "problems": _log(rng, 1, 256),
            "p": rng.choice((0.01, 0.05, 0.1, 1.0 if rng.random() < 0.3 else 0.02))}


def draw(rng):
    path = rng.choice((_draw_layer, _draw_layer, _draw_mlp, _draw_mlp, _draw_mlp, _draw_cnn, _draw_cnn, _draw_rnn,
                       _draw_sample, _draw_optimizer, _draw_pde))
    return path(rng)


# ----------------------------------------------------------------------------------------------------------- helpers
class _Owned:
    """A handle of the library, given back when the state that holds it goes."""

    def __init__(self, handle, destroy):
        self.handle = handle
        weakref.finalize(self, destroy, handle)


class _DeviceArray:
    """Memory of a model, for torch to look at; `owner` lives as long as any tensor made of it."""

    def __init__(self, owner, ptr, shape, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": shape, "typestr": typestr, "version": 2}


_context = None


def _ctx():
    """One context for the program, on the default stream."""
    global _context
    if _context is None:
        _context = B.rad_ctx_create()
    return _context


def _ints(text):
    return [int(v) for v in text.split("-")]


def _dtype(case):
    return (B.RAD_BF16, torch.bfloat16) if case.get("dtype") == "bf16" else (B.RAD_F32, torch.float32)


class _Maker:
    """Seeded inputs with the shapes and value statistics of the workloads (see synth.py)."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFF)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, device="cuda", generator=self.gen).mul_(std)

    def uniform(self, *shape):
        return torch.rand(*shape, device="cuda", generator=self.gen)

    def pixels(self, *shape):
        """uniform [0, 1) with 80 % of the entries zero"""
        x = self.uniform(*shape)
        return x.mul_(self.uniform(*shape) >= 0.8)

    def labels(self, n, classes):
        return torch.randint(0, classes, (n,), device="cuda", dtype=torch.int32, generator=self.gen)


def _training_state(case, seed, model, dtype, x, labels, params, classes):
    owner = _Owned(model, B.rad_model_destroy)
    logits = torch.as_tensor(_DeviceArray(owner, B.rad_model_logits(model), (case["batch"], classes),
                                          "<i2" if dtype == B.RAD_BF16 else "<f4"), device="cuda")
    return {"path": "train", "model": owner, "x": x, "labels": labels, "params": params,
            "logits": logits.view(torch.bfloat16) if dtype == B.RAD_BF16 else logits,
            "grads": [torch.empty(p.shape, device="cuda", dtype=torch.float32) for p in params],
            "sampling": B.make_sampling(SCHEMES[case["scheme"]], case["p"], seed + 1, 0, 0)}


# ----------------------------------------------------------------------------------------------------------- prepare
def _prepare_layer(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    dtype, tdt = _dtype(case)
    n, d, o = case["batch"], case["d_in"], case["d_out"]
    layer = B.make_layer(n, d, o, dtype=dtype, relu=case["relu"], has_bias=case["bias"])
    store = B.rad_store_create(ctx, layer, SCHEMES[case["scheme"]], case["p"])
    x = make.pixels(n, d) if dtype == B.RAD_F32 else make.normal(n, d)
    return {"path": "layer", "layer": layer, "store": _Owned(store, B.rad_store_destroy),
            "sampling": B.make_sampling(SCHEMES[case["scheme"]], case["p"], seed + 1, 0, 0),
            "x": x.to(tdt), "W": make.normal(d, o, std=d ** -0.5).to(tdt),
            "b": make.normal(o, std=0.1) if case["bias"] else None, "dy": make.normal(n, o, std=0.1).to(tdt),
            "y": torch.empty(n, o, device="cuda", dtype=tdt), "dX": torch.empty(n, d, device="cuda", dtype=tdt),
            "dW": torch.empty(d, o, device="cuda"), "db": torch.empty(o, device="cuda") if case["bias"] else None}


def _prepare_mlp(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    dtype, tdt = _dtype(case)
    dims, n = _ints(case["dims"]), case["batch"]
    model = B.rad_model_create_mlp(ctx, dtype, n, dims, case["bias"], SCHEMES[case["scheme"]], case["p"])
    if case["index_free"]:
        B.rad_model_set_index_free(ctx, model, True)
    params = []
    for d, o in zip(dims, dims[1:]):
        params.append(make.normal(d, o, std=d ** -0.5).to(tdt))
        if case["bias"]:
            params.append(make.normal(o, std=0.1))
    x = make.pixels(n, dims[0]) if dtype == B.RAD_F32 else make.normal(n, dims[0])
    return _training_state(case, seed, model, dtype, x.to(tdt), make.labels(n, dims[-1]), params, dims[-1])


def _prepare_cnn(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    ch, pool, ks, n = _ints(case["channels"]), _ints(case["pool"]), case["ksize"], case["batch"]
    model = B.rad_model_create_cnn(ctx, n, ch, pool, ks, case["hw"], case["hw"], case["classes"],
                                   SCHEMES[case["scheme"]], case["p"])
    params = []
    for ci, co in zip(ch, ch[1:]):
        params += [make.normal(ci, ks, ks, co, std=(ci * ks * ks) ** -0.5), make.normal(co, std=0.1)]
    d = ch[-1] * (case["hw"] >> sum(1 for v in pool if v)) ** 2
    params += [make.normal(d, case["classes"], std=d ** -0.5), make.normal(case["classes"], std=0.1)]
    x = make.normal(n, ch[0], case["hw"], case["hw"])
    return _training_state(case, seed, model, B.RAD_F32, x, make.labels(n, case["classes"]), params, case["classes"])


def _prepare_rnn(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    n, T, h, c = case["batch"], case["T"], case["hidden"], case["classes"]
    model = B.rad_model_create_rnn(ctx, n, T, 1, h, c, SCHEMES[case["scheme"]], case["p"])
    std = 0.001 ** 0.5
    params = [make.normal(1, h, std=std), torch.eye(h, device="cuda"), torch.zeros(h, device="cuda"),
              make.normal(h, c, std=std), torch.zeros(c, device="cuda")]
    return _training_state(case, seed, model, B.RAD_F32, make.uniform(n, T, 1), make.labels(n, c), params, c)


def _prepare_sample(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    dtype, tdt = _dtype(case)
    n, d, o = case["rows"], case["cols"], case["d_out"]
    layer = B.make_layer(n, d, o, dtype=dtype, relu=False)
    store = B.rad_store_create(ctx, layer, SCHEMES[case["scheme"]], case["p"])
    return {"path": "sample", "layer": layer, "store": _Owned(store, B.rad_store_destroy),
            "sampling": B.make_sampling(SCHEMES[case["scheme"]], case["p"], seed + 1, 0, 0),
            "x": make.normal(n, d).to(tdt), "dy": make.normal(n, o, std=1.0 / n).to(tdt),
            "dW": torch.empty(d, o, device="cuda")}


def _prepare_optimizer(case, seed):
    make = _Maker(seed)
    dtype, tdt = _dtype(case)
    counts, adam = _ints(case["counts"]), case["kind"] == "adam"
    master = [make.normal(n, std=1.0 / 64) for n in counts]
    params = [w.to(torch.bfloat16) for w in master] if dtype == B.RAD_BF16 else master
    return {"path": "optimizer", "dtype": dtype, "params": params, "master": master if dtype == B.RAD_BF16 else None,
            "grads": [make.normal(n, std=1e-3) for n in counts],
            "m": [make.normal(n, std=1e-4) for n in counts] if adam else None,
            "v": [make.uniform(n).mul_(1e-6) for n in counts] if adam else None,
            "opt": B.make_optimizer(B.RAD_ADAM if adam else B.RAD_SGD, 1e-4, 1e-5)}


def _prepare_pde(case, seed):
    ctx, make = _ctx(), _Maker(seed)
    q = case["problems"]
    grid = B.make_pde_grid(case["n"], case["steps"], PDE_D, PDE_DT)
    theta = torch.rand(q, 7, dtype=torch.float64, device="cuda", generator=make.gen) * 2 - 1
    return {"path": "pde", "grid": grid, "p": case["p"], "seed": seed + 1, "theta": theta,
            "workspace": torch.empty(B.rad_pde_workspace_bytes(ctx, grid, case["p"], q), dtype=torch.uint8, device="cuda"),
            "loss": torch.empty(q, dtype=torch.float64, device="cuda"),
            "grad": torch.empty(q, 7, dtype=torch.float64, device="cuda"),
            "stored": torch.empty(q, dtype=torch.int64, device="cuda")}


def prepare(case, seed):
    seed = int(seed)
    return {"layer": _prepare_layer, "mlp": _prepare_mlp, "cnn": _prepare_cnn, "rnn": _prepare_rnn,
            "sample": _prepare_sample, "optimizer": _prepare_optimizer, "pde": _prepare_pde}[case["path"]](case, seed)


# --------------------------------------------------------------------------------------------------------------- run
def run(state):
    s, ctx, path = state, _ctx(), state["path"]
    if path == "train":           # only enqueued, as a training loop issues its steps
        B.rad_train_step(ctx, s["model"].handle, s["sampling"], s["x"], s["labels"], s["params"], s["grads"], False)
        return {"logits": s["logits"], "grads": s["grads"]}
    if path == "layer":
        store = s["store"].handle
        B.rad_forward_sample(ctx, s["layer"], s["sampling"], s["x"], s["W"], s["b"], s["y"], store)
        B.rad_backward_dW(ctx, s["layer"], store, s["dy"], s["dW"], s["db"])
        B.rad_backward_dX(ctx, s["layer"], store, s["dy"], s["W"], s["dX"])
        return {"y": s["y"], "dW": s["dW"], "db": s["db"], "dX": s["dX"]}
    if path == "sample":
        store = s["store"].handle
        B.rad_sample_pack(ctx, s["sampling"], s["x"], store)
        B.rad_backward_dW(ctx, s["layer"], store, s["dy"], s["dW"])
        return {"dW": s["dW"]}
    if path == "optimizer":
        B.rad_optimizer_step(ctx, s["opt"], 7, s["dtype"], s["params"], s["grads"], s["m"], s["v"], s["master"])
        return {"params": s["params"], "master": s["master"], "m": s["m"], "v": s["v"]}
    B.rad_pde_gradient(ctx, s["grid"], s["theta"], s["p"], s["seed"], 0, s["workspace"], s["loss"], s["grad"], s["stored"])
    return {"loss": s["loss"], "grad": s["grad"], "stored": s["stored"]}


# -------------------------------------------------------------------------------------------------- work and tolerance
def _linear_work(case, n, dims, elem, bias, first_dx):
    """Forward, dW from the kept fraction and dX (also of the first layer if first_dx) of a stack of linear layers."""
    frac = case["p"]
    flops = nbytes = 0.0
    for l, (d, o) in enumerate(zip(dims, dims[1:])):
        flops += 2.0 * n * d * o * (1.0 + frac + (1.0 if l > 0 or first_dx else 0.0))
        nbytes += d * o * (elem + 4.0) + (8.0 * o if bias else 0.0)        # weights in, gradients out
    return flops, nbytes


def work(case):
    path = case["path"]
    elem = 2.0 if case.get("dtype") == "bf16" else 4.0
    if path == "layer":
        n, d, o = case["batch"], case["d_in"], case["d_out"]
        flops, nbytes = _linear_work(case, n, [d, o], elem, case["bias"], True)
        return {"bytes": nbytes + elem * n * (2.0 * d + 2.0 * o), "flops": flops}      # x, dy in; y, dX out
    if path == "mlp":
        n, dims = case["batch"], _ints(case["dims"])
        flops, nbytes = _linear_work(case, n, dims, elem, case["bias"], False)
        return {"bytes": nbytes + elem * n * (dims[0] + dims[-1]) + 4.0 * n, "flops": flops}
    if path == "cnn":
        n, ch, pool, size = case["batch"], _ints(case["channels"]), _ints(case["pool"]), case["hw"]
        flops, nbytes = 0.0, 4.0 * n * ch[0] * size * size
        for l, (ci, co) in enumerate(zip(ch, ch[1:])):
            w = ci * case["ksize"] ** 2 * co
            flops += 2.0 * n * size * size * w * (1.0 + case["p"] + (1.0 if l > 0 else 0.0))
            nbytes += 8.0 * (w + co)
            size = size // 2 if pool[l] else size
        d = ch[-1] * size * size
        f, b = _linear_work(case, n, [d, case["classes"]], 4.0, True, True)
        return {"bytes": nbytes + b + 4.0 * n * (1 + case["classes"]), "flops": flops + f}
    if path == "rnn":
        n, T, h, c = case["batch"], case["T"], case["hidden"], case["classes"]
        flops = 2.0 * n * h * h * (T - 1) * (2.0 + case["p"]) + 8.0 * n * h * T + 2.0 * n * h * c * (2.0 + case["p"])
        return {"bytes": 8.0 * (h * h + 2 * h + h * c + c) + 4.0 * n * (T + 1 + c), "flops": flops}
    if path == "sample":
        n, d, o = case["rows"], case["cols"], case["d_out"]
        stored = case["p"] * n * d * (elem + 2.0)                                      # written once, read once
        return {"bytes": elem * n * (d + o) + 2.0 * stored + 4.0 * d * o, "flops": 2.0 * case["p"] * n * d * o}
    if path == "optimizer":
        n = float(sum(_ints(case["counts"])))
        per = (28.0, 14.0) if case["kind"] == "adam" else (12.0, 4.0)
        return {"bytes": n * (per[0] + (2.0 if case["dtype"] == "bf16" else 0.0)), "flops": n * per[1]}
    cells = (case["n"] - 1.0) ** 2 * case["steps"] * case["problems"]
    return {"bytes": 16.0 * case["p"] * cells + 8.0 * 16 * case["problems"], "flops": 26.0 * cells}


def tolerance(case):
    """About four times what the library's results and the same sums in 64 bits differ by, over several seeds."""
    path = case["path"]
    if path == "pde":                                   # fp64 throughout
        return {"rel": 1e-11, "max": 1e-10}
    if path == "optimizer":                             # element by element; a bf16 copy may round the other way
        return {"rel": 1e-6, "max": 1e-2 if case["dtype"] == "bf16" else 1e-5}
    if path == "sample":                                # fp32 sums of the same products (7e-7)
        return {"rel": 5e-6, "max": 5e-5}
    if path == "rnn":                                   # (8e-7)
        return {"rel": 1e-5, "max": 1e-4}
    if case.get("dtype") == "bf16":
        # layer outputs, samples and gradients are rounded to bf16, and one that rounds the other way, or a ReLU bit
        # of a pre-activation at zero, is passed on (a whole step: 3e-3, one entry of a gradient as much as 0.7 of
        # its size; the calls of one layer: 1.7e-3 and 0.1)
        return {"rel": 1.2e-2, "max": 0.99} if path == "mlp" else {"rel": 7e-3, "max": 0.5}
    # fp32 sums (5e-7).  Of millions of pre-activations and pooling windows one or two lie within a rounding of a tie
    # and may fall either way, which moves a gradient by up to 2e-3 and one of its entries by 0.05.
    if path == "cnn":
        ties = case["batch"] * max(_ints(case["channels"])[1:]) * case["hw"] ** 2
    elif path == "mlp":
        ties = case["batch"] * sum(_ints(case["dims"])[1:-1])
    else:
        ties = case["batch"] * case["d_out"]
    return {"rel": 8e-3, "max": 0.2} if ties >= 200000 else {"rel": 1e-5, "max": 1e-3}
