"""The work a user of this framework has it do, as cases that can be timed and compared.

A pass is one iteration of a user's training loop: draw the minibatch (where the data is resident), take the workers'
step, offer the communication round.  The cases run from the smallest model, where a step is a few launches, to the
widest one, which fills the chip, through every family the library has: fp32 and bf16 MLPs, the small CNN, flat
parameter vectors, the first-order baselines and the data partition, with whole and ragged sizes.

A case is a flat dict:
  kind     "mlp", "cnn" (a training step), "flat" (update and round on caller-supplied g and Hz), "partition"
  dims     layer widths as text, "784-512-512-10"; flat: params = P; partition: points = n, shared = o
  k, batch, dtype ("f32" | "bf16"), fuse, probes, avg (averaging block), opt (0 AdaHessian, 1 SGD, 2 momentum)
  tau, mode ("dynamic", "fixed", "sequential"), absent (True: a third of the communications is suppressed)
  resident (points of a data set on the device the minibatches are drawn from; 0: a pool of minibatches)
  img, conv (CNN: input image "28-28-1" and channels "32-64")
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2409_09242_amd import binding as B

LR, BETA1, BETA2, EPS, ALPHA, MOMENTUM = 0.01, 0.9, 0.999, 1e-4, 0.1, 0.5
POOL = 4                       # minibatches a user's input pipeline has ready
TAKEN = 10                     # local steps that a network case's workers have behind them
DEVICE = "cuda:0"


def _mlp(name, dims, k, batch, dtype="f32", **more):
    c = {"kind": "mlp", "dims": dims, "k": k, "batch": batch, "dtype": dtype, "fuse": 0, "probes": 1, "avg": 1, "opt": 0,
         "tau": 1, "mode": "dynamic", "absent": False, "resident": 0}
    c.update(more)
    if name:
        c["name"] = name
    return c


def _cnn(name, img, conv, fc, k, batch, **more):
    return _mlp(name, fc, k, batch, kind="cnn", img=img, conv=conv, **more)


def _flat(name, params, k, **more):
    c = {"kind": "flat", "params": params, "k": k, "avg": 1, "opt": 0, "tau": 1, "mode": "dynamic", "absent": False}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest model, a round after every step: launches and latency are everything
        _mlp("tiny_mlp_round", "32-64-10", 4, 16),
        # MNIST-shaped MLP in fp32, minibatches drawn from 60000 resident points: an ordinary small training run
        _mlp("mnist_mlp_resident", "784-512-512-10", 4, 128, tau=4, resident=60000),
        # the same model under elastic averaging SGD with momentum, the baseline the method is compared with
        _mlp("mnist_mlp_momentum", "784-512-512-10", 4, 128, tau=4, opt=2, mode="fixed", absent=True),
        # CIFAR-shaped MLP in fp32, the update fused into the weight gradients, failed workers
        _mlp("cifar_mlp_fused", "3072-1024-1024-1024-10", 8, 256, tau=8, fuse=1, absent=True),
        # nothing a multiple of a tile: odd batch, widths of 4, 7 classes; defaults otherwise
        _mlp("ragged_mlp_f32", "396-1036-340-7", 5, 93, tau=2),
        # bf16 with the defaults (g and Hz stay readable) at widths that are no multiple of a tile
        _mlp("ragged_mlp_bf16", "1208-1544-776-10", 6, 200, "bf16", tau=2, avg=8),
        # the widest model: 50M parameters in each of 16 replicas, everything fused
        _mlp("wide_mlp_bf16_fused", "4096-4096-4096-4096-10", 16, 512, "bf16", tau=4, fuse=1, absent=True),
        # two Hutchinson probes a step
        _mlp("two_probes_bf16_fused", "2048-2048-2048-10", 16, 512, "bf16", tau=4, fuse=1, probes=2),
        # the two-convolution network of the paper's experiments, window averaging, a round every step
        _cnn("cnn_paper_model", "28-28-1", "32-64", "9216-128-10", 8, 64, absent=True),
        # update and round alone at 1e8 parameters in each of 16 replicas: the HBM-bound path
        _flat("update_round_1e8", 100_000_000, 16),
        # the same path on a vector that is no multiple of anything, with averaging and sequential exchanges
        _flat("update_round_ragged", 1_234_572, 7, avg=4, mode="sequential", absent=True),
        # the overlap partition of a data set of MNIST's size over 8 workers, once per run
        {"name": "partition_60000", "kind": "partition", "points": 60000, "shared": 7500, "k": 8},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi, step):
    """A width of the range: half the time any multiple of `step`, else a multiple of 128 where the range has one."""
    w = _log(rng, lo, hi)
    if hi >= 256 and rng.random() < 0.5:
        return max(128, int(round(w / 128)) * 128)
    return max(step, int(round(w / step)) * step)


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["bytes"] / 4.0e12 + w["flops"] / (5.0e14 if c.get("dtype") == "bf16" else 5.0e13) < 7e-3:
            return c


def _draw(rng):
    what = rng.choice(["tiny", "f32", "f32", "bf16", "bf16", "cnn", "flat", "flat", "partition"])
    mode = rng.choice(["dynamic", "dynamic", "fixed", "sequential"])
    common = {"tau": rng.choice([1, 2, 4, 8]), "mode": mode, "absent": rng.random() < 0.5}
    if what == "tiny":
        dims = [_width(rng, 8, 64, 4)] + [_width(rng, 8, 96, 4) for _ in range(rng.choice([1, 1, 2]))] + [rng.randint(2, 16)]
        return _mlp(None, "-".join(map(str, dims)), rng.randint(1, 16), rng.randint(4, 32), **dict(common, tau=1))
    if what in ("f32", "bf16"):
        half = what == "bf16"
        step = 8 if half else 4
        hi = 4096 if half else 2048
        dims = [_width(rng, 128, 4096 if half else 3072, step)]
        dims += [_width(rng, 96, hi, step) for _ in range(rng.choice([1, 2, 2, 3]))]
        dims += [rng.randint(2, 16)]
        opt = rng.choice([0, 0, 0, 0, 1, 2])
        probes = 1 if opt else rng.choice([1, 1, 1, 2, 3])
        fuse = 0 if opt else rng.choice([0, 1])
        avg = 1 if opt else rng.choice([1, 1, 4])
        batch = rng.choice([64, 128, 256, 512, rng.randint(17, 300)])
        return _mlp(None, "-".join(map(str, dims)), rng.randint(1, 16), batch, what, fuse=fuse, probes=probes, avg=avg, opt=opt,
                    resident=rng.choice([0, 0, 0, 20000]), **common)
    if what == "cnn":
        h, w = 2 * rng.randint(6, 16), 2 * rng.randint(6, 16)
        ch = [4 * rng.randint(2, 8), 4 * rng.randint(4, 16)][: rng.choice([1, 2, 2])]
        flat = ((h - 2 * len(ch)) // 2) * ((w - 2 * len(ch)) // 2) * ch[-1]
        return _cnn(None, "%d-%d-%d" % (h, w, rng.choice([1, 1, 3])), "-".join(map(str, ch)),
                    "%d-%d-%d" % (flat, 4 * rng.randint(8, 48), rng.randint(2, 16)), rng.randint(1, 8), rng.randint(8, 96),
                    probes=rng.choice([1, 1, 2]), **common)
    if what == "flat":
        avg = rng.choice([1, 1, 4, 32])
        opt = rng.choice([0, 0, 0, 1, 2])
        unit = max(4, avg)
        return _flat(None, int(_log(rng, 2e3, 1e8) / unit) * unit, rng.randint(1, 16), avg=avg, opt=opt, **dict(common, tau=1))
    n = int(_log(rng, 1000, 200_000))
    return {"kind": "partition", "points": n, "shared": int(n * rng.choice([0.0, 0.125, 0.25, 0.5])), "k": rng.randint(2, 16)}


# ---- shapes -----------------------------------------------------------------------------------------------------------

def _ints(text):
    return [int(t) for t in text.split("-")]


def _layers(case):
    """[(kind, offset of W, offset of b, rows, row length, used row length)] of the library's parameter layout, and P."""
    out, at = [], 0
    if case["kind"] == "cnn":
        c_in = _ints(case["img"])[2]
        for co in _ints(case["conv"]):
            row = (9 * c_in + 3) // 4 * 4
            out.append(("conv", at, at + co * row, co, row, 9 * c_in))
            at += co * row + co
            c_in = co
    dims = _ints(case["dims"])
    for a, b in zip(dims[:-1], dims[1:]):
        out.append(("linear", at, at + a * b, b, a, a))
        at += a * b + b
    return out, at


def _products(case):
    """(rows, fan-in, fan-out) of every layer's product for one worker."""
    n, out = case["batch"], []
    if case["kind"] == "cnn":
        h, w, c_in = _ints(case["img"])
        for co in _ints(case["conv"]):
            h, w = h - 2, w - 2
            out.append((n * h * w, 9 * c_in, co))
            c_in = co
    dims = _ints(case["dims"])
    return out + [(n, a, b) for a, b in zip(dims[:-1], dims[1:])]


def _round_bytes(P, k, due):
    """theta of every worker read and written, the centre read and written."""
    return due * (8.0 * P * k + 8.0 * P)


def work(case):
    k = case["k"]
    if case["kind"] == "partition":
        n, o = case["points"], case["shared"]
        return {"bytes": 4.0 * k * (o + (n - o) // k), "flops": 0.0}     # the index array written once
    state = {0: 24.0, 1: 8.0, 2: 16.0}[case["opt"]]                      # theta (m, v) read and written
    if case["kind"] == "flat":
        P = case["params"]
        given = 8.0 if case["opt"] == 0 else 4.0                         # g (and Hz) read
        return {"bytes": (state + given) * P * k + _round_bytes(P, k, 1.0 / case["tau"]), "flops": 20.0 * P * k}
    P = _layers(case)[1]
    flops = 0.0
    for i, (rows, fan_in, fan_out) in enumerate(_products(case)):
        one = 2.0 * rows * fan_in * fan_out
        if case["opt"]:
            flops += one * (2 if i == 0 else 3)                          # forward, weight gradient, data gradient
        else:
            # plain products once, their directional derivatives once per probe (the input has none)
            flops += one * ((2 + 2 * case["probes"]) if i == 0 else (3 + 6 * case["probes"]))
    img = case["kind"] == "cnn"
    sample = math.prod(_ints(case["img"])) if img else _ints(case["dims"])[0]
    x = k * case["batch"] * sample * (2.0 if case["dtype"] == "bf16" else 4.0)
    return {"bytes": state * P * k + x * (3.0 if case["resident"] else 1.0) + _round_bytes(P, k, 1.0 / case["tau"]),
            "flops": flops * k}


# ---- inputs -----------------------------------------------------------------------------------------------------------

def _gen(seed, stream):
    return torch.Generator(device=DEVICE).manual_seed((int(seed) * 1009 + stream) & 0x7FFFFFFF)


def _theta0(case, seed):
    """U(+-1/sqrt(fan-in)) per layer (flat: U(+-0.01)); padding entries of a kernel's rows are zero."""
    g = _gen(seed, 1)
    if case["kind"] == "flat":
        return (torch.rand(case["params"], generator=g, device=DEVICE) * 2 - 1) * 0.01
    layers, P = _layers(case)
    t = torch.empty(P, device=DEVICE)
    for _, wo, bo, rows, row, used in layers:
        bound = 1.0 / math.sqrt(used)
        w = (torch.rand(rows, row, generator=g, device=DEVICE) * 2 - 1) * bound
        w[:, used:] = 0.0
        t[wo:wo + rows * row] = w.reshape(-1)
        t[bo:bo + rows] = (torch.rand(rows, generator=g, device=DEVICE) * 2 - 1) * bound
    return t


def _forward(case, theta, x, margins=None):
    """Logits of one worker's samples x [n][...] in theta's type; margins: receives, per sample, how near its closest
    unit (or pooling choice) is to its kink, in units of the layer's root mean square."""
    def note(t, n):
        if margins is not None:
            r = t.abs().reshape(n, -1).amin(1) / t.square().mean().sqrt()
            margins.append(r)

    n, a = x.shape[0], x
    for i, (kind, wo, bo, rows, row, used) in enumerate(_layers(case)[0]):
        w, b = theta[wo:wo + rows * row].reshape(rows, row), theta[bo:bo + rows]
        if kind == "conv":
            h, wd, ci = a.shape[1:]
            cols = F.unfold(a.permute(0, 3, 1, 2), 3)                     # [n][ci*9][positions], entry ci*9 + tap
            cols = cols.reshape(n, ci, 9, -1).permute(0, 3, 2, 1).reshape(-1, 9 * ci)
            s = cols @ w[:, :used].t() + b
            note(s, n)
            a = torch.relu(s).reshape(n, h - 2, wd - 2, rows)
            last = _layers(case)[0][i + 1][0] != "conv"
            if last:
                m = a.permute(0, 3, 1, 2)
                if margins is not None:
                    p = F.unfold(m.reshape(-1, 1, h - 2, wd - 2), 2, stride=2).sort(1, descending=True).values
                    gap = torch.where(p[:, 0] > 0, p[:, 0] - p[:, 1], torch.ones_like(p[:, 0]))
                    margins.append(gap.reshape(n, -1).amin(1) / p.square().mean().sqrt())
                a = F.max_pool2d(m, 2).permute(0, 2, 3, 1).reshape(n, -1)
        else:
            s = a @ w.t() + b
            if i == len(_layers(case)[0]) - 1:
                return s
            note(s, n)
            a = torch.relu(s)


def _fresh(case, gen, n):
    shape = (n,) + (tuple(_ints(case["img"])) if case["kind"] == "cnn" else (_ints(case["dims"])[0],))
    # images and MNIST-shaped inputs U[0,1], the others N(0,1)
    uniform = case["kind"] == "cnn" or shape[-1] == 784
    x = torch.rand(shape, generator=gen, device=DEVICE) if uniform else torch.randn(shape, generator=gen, device=DEVICE)
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _samples(case, theta0, seed, stream, n, watch):
    """n samples.  `watch`: samples with a unit or pooling choice that 32-bit sums may put on either side of its kink
    are drawn again, since the derivative has two right values there: within 1e-5 of the layer's root mean square in
    an MLP (contractions of up to 4096), 2e-6 in the CNN (most of them 9 and 288 long)."""
    gen = _gen(seed, stream)
    near_kink = 2e-6 if case["kind"] == "cnn" else 1e-5
    x = _fresh(case, gen, n)
    if watch and case["dtype"] == "f32":
        t = theta0.double()
        bad = torch.arange(n, device=DEVICE)
        for _ in range(12):
            near = []
            for part in bad.split(64 if case["kind"] == "cnn" else 4096):
                m = []
                _forward(case, t, x[part].double(), m)
                near.append(torch.stack(m).amin(0) < near_kink)
            bad = bad[torch.cat(near)]
            if not bad.numel():
                break
            x[bad] = _fresh(case, gen, bad.numel())
    return x


def _teacher(case, seed):
    d0 = math.prod(_ints(case["img"])) if case["kind"] == "cnn" else _ints(case["dims"])[0]
    return torch.randn(d0, _ints(case["dims"])[-1], generator=_gen(seed, 2), device=DEVICE)


def _labels(teacher, x):
    """Argmax of a random linear teacher on centred inputs."""
    v = x.reshape(-1, teacher.shape[0]).float()
    return ((v - v.mean()) @ teacher).argmax(1).to(torch.int32).reshape(x.shape[0])


def _minibatches(case, seed, theta0, count):
    """(x [k][B][...], y [k][B]) pairs, the first one watched (see _samples)."""
    teacher, out = _teacher(case, seed), []
    k, n = case["k"], case["batch"]
    for j in range(count):
        x = _samples(case, theta0, seed, 10 + j, k * n, j == 0)
        out.append((x.reshape((k, n) + tuple(x.shape[1:])), _labels(teacher, x).reshape(k, n)))
    return out


def _dataset(case, seed, theta0):
    x = _samples(case, theta0, seed, 10, case["resident"], True)
    return x, _labels(_teacher(case, seed), x)


def _masks(case, seed):
    """Who communicates in each of 32 rounds; a third is suppressed, never everybody at once."""
    if not case["absent"]:
        return [None] * 32
    r = np.random.RandomState(seed & 0x7FFFFFFF)
    m = (r.rand(32, case["k"]) >= 1.0 / 3.0).astype(np.uint8)
    m[m.sum(1) == 0, 0] = 1
    return list(m)


def _config(case, seed):
    kw = dict(k=case["k"], lr=LR, beta1=BETA1, beta2=BETA2, eps=EPS, alpha=ALPHA, avg_block=case["avg"], seed=int(seed),
              optimizer=case["opt"], momentum=MOMENTUM)
    if case["kind"] == "flat":
        return B.make_config(dims=None, n_params=case["params"], **kw)
    kw.update(dims=_ints(case["dims"]), batch=case["batch"], bf16=case["dtype"] == "bf16", n_samples=case["probes"],
              fuse_update=case["fuse"])
    if case["kind"] == "cnn":
        kw.update(img=_ints(case["img"]), conv=_ints(case["conv"]), conv_avg=1)
    return B.make_config(**kw)


def _views(h, theta0, opt):
    """theta, m, v [k][P] and the centre [P] as tensors over the caller's workspace.

    dw_set_state puts a mark on the first entry of each array, the mark's place in the workspace is where the array is,
    and the entry's own value goes back: what dw_get_state copies to the host, without a copy."""
    f = h.workspace[h._ws_ptr - h.workspace.data_ptr():]
    f = f[: f.numel() // 4 * 4].view(torch.float32)
    arrays = [("theta", B.DW_S_THETA)] + ([("m", B.DW_S_M)] if opt != 1 else []) + ([("v", B.DW_S_V)] if opt == 0 else [])
    marks = [(name, what, i) for name, what in arrays for i in range(min(h.k, 2))] + [("centre", B.DW_S_CENTRE, 0)]
    for j, (_, what, i) in enumerate(marks):
        h.set_state(what, i, [1e30 * (j + 1)])
    found = {}
    step = 1 << 29
    for at in range(0, f.numel(), step):
        part = f[at:at + step]
        for p in (part.abs() > 5e29).nonzero().reshape(-1).tolist():
            found[int(round(float(part[p]) / 1e30)) - 1] = at + p
    first = float(theta0[0])
    for _, what, i in marks:
        h.set_state(what, i, [first if what in (B.DW_S_THETA, B.DW_S_CENTRE) else 0.0])
    out = {}
    for j, (name, _, i) in enumerate(marks):
        if name == "centre":
            out[name] = f[found[j]:found[j] + h.P]
        elif i == 0:
            stride = found[j + 1] - found[j] if h.k > 1 else h.P
            out[name] = torch.as_strided(f, (h.k, h.P), (stride, 1), f.storage_offset() + found[j])
    return out


def _second_moments(case, theta0, x, y, seed):
    """v after TAKEN steps, one value for each weight matrix and bias vector: the mean square of D on a minibatch.  (Rounded to
    a power of two, so that it comes out the same everywhere.)"""
    p = theta0.double().requires_grad_(True)
    (g,) = torch.autograd.grad(F.cross_entropy(_forward(case, p, x.double()), y.long()), p, create_graph=True)
    z = torch.randint(0, 2, (p.numel(),), generator=_gen(seed, 4), device=DEVICE).double() * 2 - 1
    (hz,) = torch.autograd.grad(g, p, z)
    D2 = _averaged(case, z * hz).square()
    v = np.zeros(p.numel(), dtype=np.float32)
    for _, wo, bo, rows, row, used in _layers(case)[0]:
        for at, shape, cols in ((wo, (rows, row), used), (bo, (1, rows), rows)):
            n = shape[0] * shape[1]
            mean = float(D2[at:at + n].reshape(shape)[:, :cols].mean())
            v[at:at + n].reshape(shape)[:, :cols] = (1 - BETA2 ** TAKEN) * 2.0 ** round(math.log2(max(mean, 1e-30)))
    return v


def _under_way(case, h, theta0, x, y, seed):
    """Puts the workers where a run has them after a few steps, as a restored checkpoint does: step counts and second
    moments.  (From v = 0 the very first step divides by |D| + eps alone, and the few entries whose D happens to cancel
    are thrown far away by any change of rounding; later steps divide by an average.)"""
    v = _second_moments(case, theta0, x, y, seed) if case["opt"] == 0 else None
    for i in range(h.k):
        h.set_state(B.DW_S_STEPS, i, [TAKEN])
        if v is not None:
            h.set_state(B.DW_S_V, i, v)


def prepare(case, seed):
    if case["kind"] == "partition":
        return {"case": case, "seed": int(seed), "i": 0}
    k = case["k"]
    theta0 = _theta0(case, seed)
    h = B.Handle(_config(case, seed), theta0, device=DEVICE)
    st = {"case": case, "h": h, "out": _views(h, theta0, case["opt"]), "masks": _masks(case, seed), "i": 0, "round": 0,
          "mode": {"dynamic": B.DW_DYNAMIC, "fixed": B.DW_FIXED, "sequential": B.DW_DYNAMIC | B.DW_SEQUENTIAL}[case["mode"]]}
    if case["kind"] == "flat":
        g = _gen(seed, 3)
        st["g"] = torch.randn(k, case["params"], generator=g, device=DEVICE).mul_(0.1)
        st["hz"] = torch.randn(k, case["params"], generator=g, device=DEVICE).mul_(0.1) if case["opt"] == 0 else None
        return st
    st["out"]["loss"] = torch.zeros(k, device=DEVICE)
    if case["resident"]:
        st["data"], st["labels"] = _dataset(case, seed, theta0)
        st["index"] = B.overlap_partition(case["resident"], case["resident"] // 8, k, int(seed) + 1, DEVICE)
        st["x"] = torch.empty((k, case["batch"]) + tuple(st["data"].shape[1:]), dtype=st["data"].dtype, device=DEVICE)
        st["y"] = torch.empty((k, case["batch"]), dtype=torch.int32, device=DEVICE)
        st["draws"] = int(seed) + 2
        few = case["batch"]
        _under_way(case, h, theta0, st["data"][:few], st["labels"][:few], seed)
    else:
        st["pool"] = _minibatches(case, seed, theta0, POOL)
        _under_way(case, h, theta0, st["pool"][0][0][0], st["pool"][0][1][0], seed)
    return st


def run(state):
    case = state["case"]
    i = state["i"]
    state["i"] = i + 1
    if case["kind"] == "partition":
        return B.overlap_partition(case["points"], case["shared"], case["k"], state["seed"] + i, DEVICE)
    h = state["h"]
    if case["kind"] == "flat":
        h.update_only(state["g"], state["hz"])
    else:
        if case["resident"]:
            x, y = state["x"], state["y"]
            h.draw_batch(state["data"], state["labels"], state["index"], state["draws"], x, y)
        else:
            x, y = state["pool"][i % POOL]
        h.worker_step(x, y, loss=state["out"]["loss"])
    if h.elastic_sync(state["mode"], tau=case["tau"], participate=state["masks"][state["round"] % 32]):
        state["round"] += 1
    return state["out"]


# ---- tolerances -------------------------------------------------------------------------------------------------------

def tolerance(case):
    if case["kind"] == "partition":
        return "exact"
    if case["kind"] == "flat":
        # element by element: a few roundings of an fp32 value
        return {"rel": 2e-6, "max": 2e-5}
    if case["dtype"] == "bf16":
        # one stored value in a thousand rounds to its other neighbour when a sum takes another order, and units within
        # 2e-3 of zero then switch; measured with theta0 moved by one fp32 bit at 4096 wide: m 1.9e-2 (max 1.0) after
        # one step, 3.1e-2 after two
        return {"rel": 3e-2, "max": 0.99}
    # fp32 sums in another order; on the second step, whose samples are not watched, a unit or two of the largest model
    # land on the other side of their kink, and each moves one of batch x width terms.  Measured with theta0 moved by one
    # fp32 bit: 7e-7 after the first step, m 9e-4 (max 0.3) after the second
    return {"rel": 4e-3, "max": 0.9}


# ---- the first pass in 64 bits -----------------------------------------------------------------------------------------

_M64 = (1 << 64) - 1
_GAMMA = 0x9E3779B97F4A7C15


def _mix(x):
    """SplitMix64's output function on a Python integer."""
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & _M64
    return x ^ (x >> 31)


def _signed(x):
    return x - (1 << 64) if x >> 63 else x


def _mix_t(x):
    """The same on an int64 tensor (products wrap, shifts are made logical)."""
    x = (x ^ ((x >> 30) & ((1 << 34) - 1))) * _signed(0xBF58476D1CE4E5B9)
    x = (x ^ ((x >> 27) & ((1 << 37) - 1))) * _signed(0x94D049BB133111EB)
    return x ^ ((x >> 31) & ((1 << 33) - 1))


def _stream_key(seed, i, t):
    return _mix((_mix((seed + _GAMMA * (i + 1)) & _M64) + _GAMMA * (t + 1)) & _M64)


def _counter_words(key, n):
    w = torch.arange(1, n + 1, dtype=torch.int64, device=DEVICE) * _signed(_GAMMA)
    return _mix_t(w + _signed(key))


def _rademacher(seed, i, t, P):
    words = _counter_words(_stream_key(seed, i, t), (P + 63) // 64)
    bits = (words[:, None] >> torch.arange(64, device=DEVICE)) & 1
    return bits.reshape(-1)[:P].double() * 2 - 1


def _partition(n, o, k, seed):
    keys = _counter_words(_mix(seed), n)
    perm = torch.sort(keys ^ _signed(1 << 63), stable=True).indices.to(torch.int32)   # unsigned order
    s = (n - o) // k
    return torch.stack([torch.cat([perm[:o], perm[o + j * s:o + (j + 1) * s]]) for j in range(k)])


def _first_minibatch(case, seed, theta0):
    """x, y of the first pass and v before it."""
    if not case["resident"]:
        x, y = _minibatches(case, seed, theta0, 1)[0]
        return x, y, _second_moments(case, theta0, x[0], y[0], seed) if case["opt"] == 0 else None
    data, labels = _dataset(case, seed, theta0)
    few = case["batch"]
    v = _second_moments(case, theta0, data[:few], labels[:few], seed) if case["opt"] == 0 else None
    index = _partition(case["resident"], case["resident"] // 8, case["k"], seed + 1)
    m, xs, ys = index.shape[1], [], []
    for j in range(case["k"]):
        key = _stream_key(seed + 2, j, TAKEN)
        pos = [(_mix((key + _GAMMA * (b + 1)) & _M64) * m) >> 64 for b in range(case["batch"])]
        idx = index[j].long()[torch.tensor(pos, device=DEVICE)]
        xs.append(data[idx])
        ys.append(labels[idx])
    return torch.stack(xs), torch.stack(ys), v


def _averaged(case, D):
    """Block means along fan-in of the weights' entries; window means of the convolutions'."""
    if case["kind"] == "flat":
        return D.reshape(-1, case["avg"]).mean(1, keepdim=True).expand(-1, case["avg"]).reshape(-1)
    D = D.clone()
    for kind, wo, bo, rows, row, used in _layers(case)[0]:
        if kind == "conv":
            w = D[wo:bo].reshape(rows, row)
            w[:, :used] = w[:, :used].reshape(rows, 9, -1).mean(1, keepdim=True).expand(-1, 9, -1).reshape(rows, used)
        elif case["avg"] > 1:
            w = D[wo:bo].reshape(-1, case["avg"])
            w[:] = w.mean(1, keepdim=True)
    return D


def exact(case, seed):
    if case["kind"] == "partition":
        return _partition(case["points"], case["shared"], case["k"], int(seed))
    k, flat = case["k"], case["kind"] == "flat"
    cfg = _config(case, seed)
    theta0 = _theta0(case, seed)
    start = theta0.double()
    out = {"theta": [], "m": [], "v": [], "loss": []}
    if flat:
        g_all = torch.randn(k, case["params"], generator=(gen := _gen(seed, 3)), device=DEVICE).mul_(0.1)
        hz_all = torch.randn(k, case["params"], generator=gen, device=DEVICE).mul_(0.1) if case["opt"] == 0 else None
    else:
        x, y, v0 = _first_minibatch(case, seed, theta0)
        v0 = None if v0 is None else torch.from_numpy(v0).to(DEVICE).double()
    taken = 0 if flat else TAKEN
    probes = 1 if flat else case["probes"]
    # constants as the configuration holds them, in fp32
    lr, b1, b2, eps, alpha = cfg.lr, cfg.beta1, cfg.beta2, cfg.eps, cfg.alpha
    for i in range(k):
        if flat:
            g = g_all[i].double()
        else:
            p = start.clone().requires_grad_(True)
            loss = F.cross_entropy(_forward(case, p, x[i].double()), y[i].long())
            out["loss"].append(loss.detach())
            second = case["opt"] == 0
            (g,) = torch.autograd.grad(loss, p, create_graph=second)
        if case["opt"] == 0:
            D = 0.0
            for j in range(probes):
                z = _rademacher(int(seed), i, taken * probes + j, start.numel())
                if flat:
                    hz = hz_all[i].double()
                else:
                    (hz,) = torch.autograd.grad(g, p, z, retain_graph=j + 1 < probes)
                D = D + _averaged(case, z * hz)
            D = D / probes
            g = g.detach()
            m, v = (1 - b1) * g, (1 - b2) * D * D + (0.0 if flat else b2 * v0)
            out["m"].append(m)
            out["v"].append(v)
            step = (m / (1 - b1 ** (taken + 1))) / ((v / (1 - b2 ** (taken + 1))).sqrt() + eps)
        else:
            step = g.detach()
            if case["opt"] == 2:
                out["m"].append(step)
        out["theta"].append(start - lr * step)
    centre = start.clone()
    if case["tau"] == 1:                       # the first round: no history yet, so every weight is alpha
        mask = _masks(case, seed)[0]
        move, seq = torch.zeros_like(start), case["mode"] == "sequential"
        for i in range(k):
            if mask is not None and not mask[i]:
                continue
            d = out["theta"][i] - (centre if seq else start)
            out["theta"][i] = out["theta"][i] - alpha * d
            if seq:
                centre = centre + alpha * d
            else:
                move += alpha * d
        centre = centre + move
    res = {n: torch.stack(v) for n, v in out.items() if v}
    res["centre"] = centre
    return res
