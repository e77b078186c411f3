"""The workloads this framework's speed is measured on.

A case is one pass of what a training program has the library do: an SMA
iteration (cb_step then cb_sync) of k learners, a synchronisation of replicas
with the program's own gradients (cb_sma_apply), or one layer of a learning
task on the program's buffers (a convolution or a batch norm, forward and
backward, all learners in one call).

listed() gives the named cases, draw() more of the same ranges, prepare()
what a program holds before the call, run() the call, work() the bytes and
operations it cannot do without, tolerance() how far two correct fp32
implementations may be apart, and exact() the same results in float64 from
plain torch.
"""
from __future__ import annotations

import ctypes
import math

import torch
import torch.nn.functional as F
from torch.utils.flop_counter import FlopCounterMode

import paper_1901_02244_amd as cb

LR, MOMENTUM = 0.01, 0.9


def _f32(v):
    return ctypes.c_float(v).value


# ------------------------------------------------------------------- cases
def _train(arch, k, b, c, h, classes, mu_l=0.0, name=None):
    d = {"kind": "train", "arch": arch, "k": k, "b": b, "in_c": c, "h": h, "classes": classes,
         "learner_momentum": mu_l}
    return {"name": name, **d} if name else d


def _sma(arch, k, mu_l=0.0, name=None):
    d = {"kind": "sma", "arch": arch, "k": k, "learner_momentum": mu_l}
    return {"name": name, **d} if name else d


def _conv(k, b, ci, h, co, r, stride, pad, relu=False, bias=False, name=None):
    d = {"kind": "conv", "k": k, "b": b, "ci": ci, "h": h, "co": co, "r": r, "stride": stride,
         "pad": pad, "relu": relu, "bias": bias}
    return {"name": name, **d} if name else d


def _bn(k, b, c, h, name=None):
    # without the ReLU: one more or less rounding moves a few of its decisions,
    # and with each a whole element of dx (the training cases have it)
    d = {"kind": "bn", "k": k, "b": b, "c": c, "h": h}
    return {"name": name, **d} if name else d


def listed():
    return [
        # the smallest job: two LeNet learners of four images, where launches
        # and latency count
        _train("lenet5", 2, 4, 1, 28, 10, name="train_lenet_k2_b4"),
        # LeNet with enough learners that half of the chip has an image
        _train("lenet5", 8, 16, 1, 28, 10, name="train_lenet_k8_b16"),
        # one ResNet-32 learner: where the learner tuner starts from
        _train("resnet32", 1, 16, 3, 32, 10, name="train_resnet32_k1_b16"),
        # the usual ResNet-32 job (the benchmark's headline)
        _train("resnet32", 4, 32, 3, 32, 10, name="train_resnet32_k4_b32"),
        # ResNet-32 with the many small learners the method is meant for
        _train("resnet32", 32, 16, 3, 32, 10, name="train_resnet32_k32_b16"),
        # ImageNet-sized training, the largest model
        _train("resnet50", 2, 32, 3, 224, 1000, name="train_resnet50_k2_b32"),
        # the synchronisation alone at the largest size: 25.6M parameters, 32
        # replicas, past every cache
        _sma("resnet50", 32, name="sma_resnet50_k32"),
        # the same for a small model, with momentum on the learners and a
        # parameter count that is no multiple of four: latency bound
        _sma("resnet32", 8, 0.9, name="sma_resnet32_k8_momentum"),
        # single layers, forward and backward: ResNet-50's 3x3 and 1x1
        # convolutions in the middle of the network
        _conv(2, 32, 128, 28, 128, 3, 1, 1, name="conv3x3_128_28_k2_b32"),
        _conv(2, 32, 256, 14, 1024, 1, 1, 0, name="conv1x1_256_1024_14_k2_b32"),
        # a ragged strided layer with bias and ReLU: no size a multiple of a
        # tile, few images
        _conv(3, 5, 52, 45, 74, 3, 2, 1, True, True, name="conv3x3s2_ragged_k3_b5"),
        # a batch norm over large planes
        _bn(2, 32, 256, 56, name="bn_256_56_k2_b32"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("lenet", "resnet32", "resnet32", "resnet50", "sma", "conv", "conv", "conv",
                       "bn"))
    if kind == "lenet":
        k, b = _log_int(rng, 1, 24), _log_int(rng, 2, 48)
        c, h = rng.choice(((1, 28), (1, 28), (1, 28), (3, 32), (1, 20)))
        return _train("lenet5", k, b, c, h, rng.choice((10, 10, 26, 62)),
                      rng.choice((0.0, 0.0, 0.9)))
    if kind == "resnet32":
        # up to 1024 images a step; eight or more per learner, since a
        # learner's norms take their statistics from its own images
        k = _log_int(rng, 1, 64)
        b = _log_int(rng, 8, max(8, min(64, 1024 // k)))
        return _train("resnet32", k, b, 3, rng.choice((32, 32, 32, 24, 40)), rng.choice((10, 100)),
                      rng.choice((0.0, 0.0, 0.9)))
    if kind == "resnet50":
        k = rng.choice((1, 1, 2, 3))
        b = _log_int(rng, 8, 64 // k)
        return _train("resnet50", k, b, 3, rng.choice((160, 192, 224)), rng.choice((200, 1000)))
    if kind == "sma":
        arch = rng.choice(("lenet5", "resnet32", "resnet50"))
        k = _log_int(rng, 1, 24 if arch == "resnet50" else 64)
        return _sma(arch, k, rng.choice((0.0, 0.0, 0.9)))
    if kind == "bn":
        k, b = _log_int(rng, 1, 8), _log_int(rng, 4, 48)
        h = _log_int(rng, 7, 112)
        c = _log_int(rng, 16, max(16, min(2048, 2 * 32 * 256 * 3136 // (k * b * h * h))))
        return _bn(k, b, c, h)
    # a convolution: up to about 60 GFLOP forward
    r = rng.choice((1, 1, 3, 3, 3, 5, 7))
    stride = rng.choice((1, 1, 2))
    k, b = _log_int(rng, 1, 8), _log_int(rng, 1, 48)
    h = max(r, _log_int(rng, 7, 112))
    ci = _log_int(rng, 3, 512)
    per = 2.0 * k * b * (h / stride) ** 2 * ci * r * r
    co = _log_int(rng, 6, max(6, min(1024, int(6e10 / per))))
    if rng.random() < 0.5:  # the widths that networks use
        ci, co = max(16, ci // 16 * 16), max(16, co // 16 * 16)
    return _conv(k, b, ci, h, co, r, stride, rng.choice((r // 2, r // 2, 0)), rng.random() < 0.3,
                 rng.random() < 0.3)


# ----------------------------------------- the networks, for shapes and exact()
def _net(arch, x, classes, take):
    """Logits of the network on x; take(kind, *shape) hands out its
    parameters in the library's order."""

    def conv(x, co, r, st=1, pad=0, bias=False):
        w = take("w", co, x.shape[1], r, r)
        return F.conv2d(x, w, take("b", co) if bias else None, st, pad)

    def bn(x):
        return F.batch_norm(x, None, None, take("gamma", x.shape[1]), take("b", x.shape[1]), True,
                            0.0, 1e-5)

    def fc(x, co):
        return F.linear(x, take("w", co, x.shape[1]), take("b", co))

    if arch == "lenet5":
        x = F.max_pool2d(F.relu(conv(x, 6, 5, 1, 2, True)), 2)
        x = F.max_pool2d(F.relu(conv(x, 16, 5, 1, 0, True)), 2).flatten(1)
        return fc(F.relu(fc(F.relu(fc(x, 120)), 84)), classes)
    if arch == "resnet32":
        x = F.relu(bn(conv(x, 16, 3, 1, 1)))
        for stage in range(3):
            for i in range(5):
                st = 2 if stage and not i else 1
                a = F.relu(bn(conv(x, 16 << stage, 3, st, 1)))
                a = bn(conv(a, 16 << stage, 3, 1, 1))
                if st == 2:
                    x = F.pad(x[:, :, ::2, ::2], (0, 0, 0, 0, 0, a.shape[1] - x.shape[1]))
                x = F.relu(a + x)
    else:
        x = F.max_pool2d(F.relu(bn(conv(x, 64, 7, 2, 3))), 3, 2, 1)
        for stage, depth in enumerate((3, 4, 6, 3)):
            w = 64 << stage
            for i in range(depth):
                st = 2 if stage and not i else 1
                a = F.relu(bn(conv(x, w, 1, st)))
                a = F.relu(bn(conv(a, w, 3, 1, 1)))
                a = bn(conv(a, 4 * w, 1))
                if not i:
                    x = bn(conv(x, 4 * w, 1, st))
                x = F.relu(a + x)
    return fc(x.mean(dim=(2, 3)), classes)


def _tensors(arch, in_c, h, classes):
    """[(kind, shape)] of the network's parameters."""
    got = []

    def take(kind, *shape):
        got.append((kind, shape))
        return torch.empty(shape, device="meta")

    _net(arch, torch.empty(2, in_c, h, h, device="meta"), classes, take)
    return got


# the smallest images of each network, for the synchronisation alone
SMA_IMAGE = {"lenet5": (1, 28, 10), "resnet32": (3, 32, 10), "resnet50": (3, 32, 1000)}


def _shape_of(case):
    if case["kind"] == "sma":
        return SMA_IMAGE[case["arch"]]
    return case["in_c"], case["h"], case["classes"]


def _params(case):
    return sum(math.prod(s) for _, s in _tensors(case["arch"], *_shape_of(case)))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _train_inputs(case, seed):
    """Central model (He-normal, with the norms and biases near their
    start), its previous value, replicas scattered around it as in the middle
    of training, N(0, 1) images and uniform labels."""
    g = _gen(seed)
    k, n = case["k"], case["k"] * case["b"]
    c, h, classes = _shape_of(case)
    z, sd = [], []
    for kind, shape in _tensors(case["arch"], c, h, classes):
        m = math.prod(shape)
        s = math.sqrt(2.0 / math.prod(shape[1:])) if kind == "w" else 0.1
        z.append(_randn(g, m) * s + (1.0 if kind == "gamma" else 0.0))
        sd.append(torch.full((m,), s, device="cuda"))
    z, sd = torch.cat(z), torch.cat(sd)
    zp = z + 0.01 * sd * _randn(g, z.numel())
    w = z + 0.05 * sd * _randn(g, k, z.numel())
    x = _randn(g, n, c, h, h)
    y = torch.randint(classes, (n,), generator=g, device="cuda", dtype=torch.int32)
    return z, zp, w, x, y


def _sma_inputs(case, seed):
    g = _gen(seed)
    p, k = _params(case), case["k"]
    z = 0.05 * _randn(g, p)
    zp = z + 0.001 * _randn(g, p)
    return z, zp, g


def _conv_inputs(case, seed):
    g = _gen(seed)
    k, n, ci, h, co, r = (case[q] for q in ("k", "b", "ci", "h", "co", "r"))
    n *= k
    ho = (h + 2 * case["pad"] - r) // case["stride"] + 1
    nw = co * ci * r * r
    x = _randn(g, n, ci, h, h)
    w = _randn(g, k, nw + (co if case["bias"] else 0)) * math.sqrt(2.0 / (ci * r * r))
    dy = _randn(g, n, co, ho, ho) / math.sqrt(n * ho * ho / k)
    return x, w, dy, nw, ho


def _bn_inputs(case, seed):
    g = _gen(seed)
    k, b, c, h = (case[q] for q in ("k", "b", "c", "h"))
    x = _randn(g, k * b, c, h, h) * (0.5 + torch.rand(c, 1, 1, generator=g, device="cuda"))
    x += _randn(g, c, 1, 1)
    p = 0.1 * _randn(g, k, 2 * c)
    p[:, :c] += 1.0
    dy = _randn(g, k * b, c, h, h) / math.sqrt(b * h * h)
    return x, p, dy


def _dx_ok(case):
    """The library has no input gradient for the first-layer filters."""
    return (case["r"], case["stride"]) in ((1, 1), (1, 2), (3, 1), (3, 2), (5, 1))


# ----------------------------------------------------------------- prepare
def _context(case, z, zp, w):
    k = case["k"]
    c, h, classes = _shape_of(case)
    m = cb.model(case["arch"], c, h, h, classes, learner_momentum=case["learner_momentum"])
    ctx = cb.Context(m, k, case.get("b", 1), 1.0 / k, LR, MOMENTUM, z.cpu().numpy())
    P, Pp = ctx.P, (ctx.P + 63) // 64 * 64
    # the parameter state opens the workspace: replicas, gradients, z, z_prev
    # (rows of P parameters padded to a multiple of 64)
    f = ctx.workspace[:(2 * k + 2) * Pp * 4].view(torch.float32)
    views = {"replicas": f[:k * Pp].view(k, Pp)[:, :P],
             "central": f[2 * k * Pp:2 * k * Pp + P]}
    if w is not None:
        ctx.cb_set_state(w.cpu().numpy(), z.cpu().numpy(), zp.cpu().numpy())
    return ctx, views, f[2 * k * Pp + Pp:2 * k * Pp + Pp + P]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        z, zp, w, x, y = _train_inputs(case, seed)
        ctx, views, _ = _context(case, z, zp, w)
        return {"kind": kind, "ctx": ctx, "x": x, "y": y, "out": views}
    if kind == "sma":
        z, zp, g = _sma_inputs(case, seed)
        ctx, views, zprev = _context(case, z, zp, None)
        zprev.copy_(zp)
        k, P = case["k"], ctx.P
        grads = torch.empty(k, P, device="cuda")
        for j in range(k):  # replica by replica: the largest state is 3 GB
            views["replicas"][j].copy_(z + 0.01 * _randn(g, P))
            grads[j] = 0.05 * _randn(g, P)
        return {"kind": kind, "ctx": ctx, "grads": grads, "out": views}
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "conv":
        x, w, dy, nw, ho = _conv_inputs(case, seed)
        geo = tuple(case[q] for q in ("k", "b", "ci", "h", "h", "co", "r", "stride", "pad"))
        n = cb.lib().cb_test_conv_scratch_bytes(*geo)
        scratch = torch.empty(n, dtype=torch.uint8, device="cuda")
        out = {"y": torch.empty_like(dy), "grads": torch.zeros_like(w)}
        if _dx_ok(case):
            out["dx"] = torch.empty_like(x)
        args = (*geo, int(case["relu"]), int(case["bias"]), x.data_ptr(), w.data_ptr(),
                w.shape[1], out["y"].data_ptr(), None, dy.data_ptr(),
                out["dx"].data_ptr() if "dx" in out else None, out["grads"].data_ptr(),
                scratch.data_ptr(), n, stream)
        return {"kind": kind, "args": args, "hold": (x, w, dy, scratch), "out": out}
    x, p, dy = _bn_inputs(case, seed)
    k, b, c, h = (case[q] for q in ("k", "b", "c", "h"))
    n = cb.lib().cb_test_bn_scratch_bytes(k, b, c, h, h)
    scratch = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = {"y": torch.empty_like(x), "mean": torch.empty(k, c, device="cuda"),
           "istd": torch.empty(k, c, device="cuda"), "dx": torch.empty_like(x),
           "grads": torch.zeros_like(p)}
    fwd = (k, b, c, h, h, 0, x.data_ptr(), p.data_ptr(), 2 * c, out["y"].data_ptr(),
           out["mean"].data_ptr(), out["istd"].data_ptr(), scratch.data_ptr(), n, stream)
    bwd = (k, b, c, h, h, x.data_ptr(), None, 0, dy.data_ptr(), p.data_ptr(), 2 * c,
           out["mean"].data_ptr(), out["istd"].data_ptr(), out["dx"].data_ptr(),
           out["grads"].data_ptr(), scratch.data_ptr(), n, stream)
    return {"kind": kind, "fwd": fwd, "bwd": bwd, "hold": (x, p, dy, scratch), "out": out}


def _ok(rc):
    if rc:
        raise RuntimeError(f"the library returned {rc}")


def run(state):
    kind = state["kind"]
    if kind == "train":
        state["ctx"].cb_step(state["x"], state["y"])
        state["ctx"].cb_sync()
    elif kind == "sma":
        state["ctx"].cb_sma_apply(state["grads"])
    elif kind == "conv":
        _ok(cb.lib().cb_test_conv(*state["args"]))
    else:
        _ok(cb.lib().cb_test_bn_fwd(*state["fwd"]))
        _ok(cb.lib().cb_test_bn_bwd(*state["bwd"]))
    return state["out"]


# -------------------------------------------------------------------- work
def _net_flops(arch, in_c, h, classes):
    """Operations of one image's forward pass, and of its first layer's."""
    with FlopCounterMode(display=False) as f:
        _net(arch, torch.empty(1, in_c, h, h, device="meta"), classes,
             lambda kind, *shape: torch.empty(shape, device="meta"))
    first = {"lenet5": 6 * 25, "resnet32": 16 * 9, "resnet50": 64 * 49 / 4}[arch] * in_c * h * h
    return f.get_total_flops(), 2.0 * first


def work(case):
    kind, k = case["kind"], case["k"]
    if kind == "conv":
        b, ci, h, co, r = (case[q] for q in ("b", "ci", "h", "co", "r"))
        ho = (h + 2 * case["pad"] - r) // case["stride"] + 1
        macs = k * b * ho * ho * co * ci * r * r
        nx, ny, nw = k * b * ci * h * h, k * b * co * ho * ho, k * co * ci * r * r
        dx = _dx_ok(case)
        # read x, w, dy; write y, dw and dx
        return {"bytes": 4.0 * (nx * (2 if dx else 1) + 2 * ny + 2 * nw),
                "flops": 2.0 * macs * (3 if dx else 2)}
    if kind == "bn":
        # read x and dy, write y and dx
        return {"bytes": 16.0 * k * case["b"] * case["c"] * case["h"] ** 2, "flops": 0.0}
    P = _params(case)
    # replicas and gradients read, replicas written, z and z_prev both ways,
    # the learners' previous values both ways
    sync = 4.0 * P * (3 * k + 4 + (2 * k if case["learner_momentum"] else 0))
    if kind == "sma":
        return {"bytes": sync, "flops": 0.0}
    c, h, classes = _shape_of(case)
    n = k * case["b"]
    flops, first = _net_flops(case["arch"], c, h, classes)
    # images and labels in, the gradients out; three contractions a layer but
    # no input gradient for the first
    return {"bytes": sync + 4.0 * (n * (c * h * h + 1) + k * P),
            "flops": n * (3.0 * flops - first)}


# --------------------------------------------------------------- tolerance
def tolerance(case):
    """About four times what the library's results are from float64 (measured
    on two seeds of the listed cases and of 14 drawn ones)."""
    kind = case["kind"]
    if kind == "sma":
        return {"rel": 2e-7, "max": 1e-6}  # 4.3e-8, 1.7e-7
    if kind == "bn":
        return {"rel": 3e-7, "max": 2e-6}  # 5.7e-8, 2.9e-7
    if kind == "conv":
        # 2e-8 sqrt(K) for a contraction of K steps, 7e-7 at most at K = 1152
        # (max 5.6e-6)
        rel = max(3e-6, 8e-8 * math.sqrt(max(case["ci"], case["co"])) * case["r"])
        return {"rel": rel, "max": 15 * rel}
    # Updated weights.  A ReLU or max-pool decision within fp32 rounding of
    # its turning point may go either way, and moves a learner's gradient by up
    # to 3e-2 in a tensor: ResNet-32's replicas were 2.7e-8 (no such decision)
    # to 9.2e-6 off (max 1.2e-3), ResNet-50's, with hundreds of them, 9e-5 to
    # 2e-4 (max 2.4e-2).  LeNet's were 3.7e-8 off (max 2.1e-7) with none, and
    # about one image in 4000 has one.
    return {"lenet5": {"rel": 1e-5, "max": 1e-3}, "resnet32": {"rel": 4e-5, "max": 1e-2},
            "resnet50": {"rel": 6e-4, "max": 0.1}}[case["arch"]]


# ------------------------------------------------------------------- exact
def _sync64(case, w, wp, grads, z, zp):
    """Algorithm 1's synchronisation in float64."""
    al, lr, mu, ml = (_f32(v) for v in (1.0 / case["k"], LR, MOMENTUM, case["learner_momentum"]))
    s = torch.zeros_like(z)
    out = torch.empty_like(w)
    for j in range(case["k"]):
        c = al * (w[j] - z)
        out[j] = w[j] - lr * grads[j] - c + ml * (w[j] - wp[j])
        s += c
    return out, z + s + mu * (z - zp)


def exact(case, seed):
    kind, k = case["kind"], case["k"]
    if kind == "train":
        z, zp, w, x, y = (t.double() if t.is_floating_point() else t.long()
                          for t in _train_inputs(case, seed))
        b, grads = case["b"], torch.empty_like(w)
        for j in range(k):
            leaf, at = w[j].clone().requires_grad_(), [0]

            def take(_, *shape):
                at[0] += math.prod(shape)
                return leaf[at[0] - math.prod(shape):at[0]].view(shape)

            xs, ys = x[j * b:(j + 1) * b], y[j * b:(j + 1) * b]
            loss = F.cross_entropy(_net(case["arch"], xs, case["classes"], take), ys)
            grads[j], = torch.autograd.grad(loss, leaf)
        out, z1 = _sync64(case, w, w, grads, z, zp)
        # which way ResNet-32's few undecided ReLUs go (see tolerance()) is
        # not for float64 to say
        return {"replicas": None if case["arch"] == "resnet32" else out, "central": z1}
    if kind == "sma":
        z, zp, g = _sma_inputs(case, seed)
        P = z.numel()
        w, grads = [torch.empty(k, P, dtype=torch.float64, device="cuda") for _ in range(2)]
        for j in range(k):
            w[j] = z + 0.01 * _randn(g, P)
            grads[j] = 0.05 * _randn(g, P)
        # the learners' previous values start as the initial central model
        out, z1 = _sync64(case, w, z.double().expand(k, P), grads, z.double(), zp.double())
        return {"replicas": out, "central": z1}
    if kind == "conv":
        x, w, dy, nw, _ = _conv_inputs(case, seed)
        ci, co, r, b = (case[q] for q in ("ci", "co", "r", "b"))
        ys, dws, dxs = [], [], []
        for j in range(k):
            xj = x[j * b:(j + 1) * b].double().requires_grad_()
            wj = w[j, :nw].double().view(co, ci, r, r).requires_grad_()
            bj = (w[j, nw:].double() if case["bias"] else torch.zeros(co, device="cuda").double())
            bj.requires_grad_()
            yj = F.conv2d(xj, wj, bj, case["stride"], case["pad"])
            gx, gw, gb = torch.autograd.grad(yj, (xj, wj, bj), dy[j * b:(j + 1) * b].double())
            ys.append((F.relu(yj) if case["relu"] else yj).detach())
            dxs.append(gx)
            dws.append(torch.cat([gw.flatten(), gb]) if case["bias"] else gw.flatten())
        out = {"y": torch.cat(ys), "grads": torch.stack(dws)}
        if _dx_ok(case):
            out["dx"] = torch.cat(dxs)
        return out
    x, p, dy = _bn_inputs(case, seed)
    b, c, n = case["b"], case["c"], case["b"] * case["h"] ** 2
    out = {q: [] for q in ("y", "mean", "istd", "dx", "grads")}
    for j in range(k):
        xj, dj = x[j * b:(j + 1) * b].double(), dy[j * b:(j + 1) * b].double()
        ga, be = (p[j, q * c:(q + 1) * c].double().view(c, 1, 1) for q in (0, 1))
        mean = xj.mean(dim=(0, 2, 3), keepdim=True)[0]
        istd = 1.0 / (((xj - mean) ** 2).mean(dim=(0, 2, 3), keepdim=True)[0] + 1e-5).sqrt()
        xh = (xj - mean) * istd
        yj = ga * xh + be
        db, dg = (t.sum(dim=(0, 2, 3)) for t in (dj, dj * xh))
        dxj = ga * istd * (dj - db.view(c, 1, 1) / n - xh * dg.view(c, 1, 1) / n)
        for q, v in (("y", yj), ("mean", mean.flatten()), ("istd", istd.flatten()), ("dx", dxj),
                     ("grads", torch.cat([dg, db]))):
            out[q].append(v)
    return {q: torch.cat(v) if q in ("y", "dx") else torch.stack(v) for q, v in out.items()}
