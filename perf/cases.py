"""The work that a user of this library has it do, as cases that can be timed.

Training steps and epochs on Random Prototypes data (one random ±1 prototype
per class, every bit of a sample flipped with probability ``flip``) at the
sizes of the workloads in ``paper_2412_00119_amd/synth.py`` and of the paper's
own two-layer networks (1000 inputs, widths 525 and 2025, the group-size
rule), inference from one pattern to a whole held-out set, and the input side
(feature medians, median binarisation, the ±1 expansion layer).  The flip
probabilities are high enough that training does not end within the passes of
a measurement: like in the paper's setting (1000 inputs, flip 0.44) patterns
stay in M.

Every output is a whole number (or a quotient of two of them), so every
tolerance is "exact".
"""
import math
import random

import torch

from paper_2412_00119_amd import bmlp as B

DEV = "cuda"
R = 0.25      # robustness
P_R = 0.5     # reinforcement probability of the first epoch


def listed():
    return [
        # The smallest step: one 784 -> 256 layer, two tiles of work; launches and host time count.
        {"name": "step-784-256-b128", "kind": "step", "k0": 784, "k": 256, "layers": 1, "classes": 10, "bound": 15,
         "group": 64, "batch": 128, "sets": 64, "flip": 0.43},
        # The paper's Random Prototypes setting: 1000 inputs, two layers of 525, batch 100, group size by its rule
        # (105): odd widths, rows that are not 16-byte multiples, 8-bit hidden weights.
        {"name": "step-1000-525x2-b100", "kind": "step", "k0": 1000, "k": 525, "layers": 2, "classes": 10, "bound": 127,
         "group": 0, "batch": 100, "sets": 100, "flip": 0.44},
        # The paper's wide layers (2025, group size 81) with more classes, a bound that is not 2^m - 1 and a batch
        # that is no multiple of a tile.
        {"name": "step-1000-2025x3-b500", "kind": "step", "k0": 1000, "k": 2025, "layers": 3, "classes": 37, "bound": 101,
         "group": 0, "batch": 500, "sets": 40, "flip": 0.42},
        # One epoch over a device-resident training set of FashionMNIST's size, as a training program calls it.
        {"name": "epoch-784-1024x2-b256", "kind": "epoch", "k0": 784, "k": 1024, "layers": 2, "classes": 10, "bound": 127,
         "group": 64, "batch": 256, "sets": 234, "flip": 0.43},
        # An ordinary step at CIFAR-10's input size.
        {"name": "step-3072-2048x3-b512", "kind": "step", "k0": 3072, "k": 2048, "layers": 3, "classes": 10, "bound": 127,
         "group": 64, "batch": 512, "sets": 64, "flip": 0.475},
        # The benchmark workload's step.
        {"name": "step-3072-4096x4-b1024", "kind": "step", "k0": 3072, "k": 4096, "layers": 4, "classes": 100, "bound": 31,
         "group": 64, "batch": 1024, "sets": 48, "flip": 0.4},
        # The largest step: eight 8192-wide layers, 1000 classes, every pattern in M.
        {"name": "step-8192-8192x8-b4096", "kind": "step", "k0": 8192, "k": 8192, "layers": 8, "classes": 1000, "bound": 63,
         "group": 64, "batch": 4096, "sets": 4, "flip": 0.3},
        # Serving: the local outputs of every layer for one pattern (latency).
        {"name": "forward-3072-4096x4-n1", "kind": "forward", "k0": 3072, "k": 4096, "layers": 4, "classes": 100, "bound": 31,
         "group": 64, "batch": 1, "flip": 0.3},
        # Serving in batches with many classes.
        {"name": "forward-8192-8192x8-n256", "kind": "forward", "k0": 8192, "k": 8192, "layers": 8, "classes": 1000, "bound": 63,
         "group": 64, "batch": 256, "flip": 0.3},
        # Evaluation of a held-out set of 10 000 with the early-exit rule.
        {"name": "eval-3072-4096x4-n10000", "kind": "eval", "k0": 3072, "k": 4096, "layers": 4, "classes": 100, "bound": 31,
         "group": 64, "batch": 10000, "flip": 0.4},
        # A training set of FashionMNIST's size made binary: the median of every feature, then the bits.
        {"name": "binarize-784-n60000", "kind": "binarize", "k0": 784, "batch": 60000},
        # The fixed random ±1 expansion layer on integer features.
        {"name": "expand-784-3072-n10000", "kind": "expand", "raw": 784, "k0": 3072, "batch": 10000},
    ]


def _log(rng, lo, hi):
    """A whole number spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(("step", "step", "step", "epoch", "forward", "eval", "binarize", "expand"))
    if kind == "binarize":
        return {"kind": kind, "k0": _log(rng, 100, 4096), "batch": _log(rng, 500, 50000)}
    if kind == "expand":
        return {"kind": kind, "raw": _log(rng, 60, 2000), "k0": _log(rng, 256, 4096), "batch": _log(rng, 100, 10000)}
    layers = rng.randint(1, 5)
    ragged = rng.random() < 0.4   # the group-size rule on a width with a divisor in its range, else groups of 64
    k = rng.randint(75, 105) * _log(rng, 3, 40) if ragged else 64 * _log(rng, 4, 64)
    case = {"kind": kind, "k0": _log(rng, 200, 4096), "k": k, "layers": layers, "classes": _log(rng, 5, 400),
            "bound": rng.choice((7, 15, 31, 63, 101, 127)), "group": 0 if ragged else 64}
    if kind == "step":
        case.update(batch=_log(rng, 30, 2048), sets=16, flip=0.44)
    elif kind == "epoch":
        case.update(k=k if k <= 2048 else 64 * rng.randint(8, 32), layers=min(layers, 3), batch=_log(rng, 64, 512),
                    sets=rng.randint(20, 60), flip=0.44)
        if case["k"] != k:
            case["group"] = 64
    else:
        case.update(batch=_log(rng, 1, 1024) if kind == "forward" else _log(rng, 1000, 10000), flip=0.4)
    return case


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _samples(case, net, n, gen):
    """Bit rows and labels of n samples; made in pieces to bound the memory of their ±1 form."""
    k0, c = case["k0"], case["classes"]
    protos = torch.randint(0, 2, (c, k0), generator=gen, device=DEV, dtype=torch.int8) * 2 - 1
    y = torch.randint(0, c, (n,), generator=gen, device=DEV, dtype=torch.int32)
    xs = []
    for i in range(0, n, 16384):
        p = protos[y[i:i + 16384].long()]
        flip = torch.rand(p.shape, generator=gen, device=DEV) < case["flip"]
        xs.append(net.pack(torch.where(flip, -p, p)))
    return torch.cat(xs), y


def _features(case, width, gen):
    """int8 features with a scale of their own and a share of zeros, as quantised activations have."""
    n = case["batch"]
    scale = torch.rand(width, generator=gen, device=DEV) * 40 + 5
    x = torch.empty((n, width), dtype=torch.int8, device=DEV)
    for i in range(0, n, 16384):
        v = torch.randn((min(16384, n - i), width), generator=gen, device=DEV) * scale
        x[i:i + 16384] = torch.where(v < -20, 0.0, v).clamp_(-128, 127).to(torch.int8)
    return x


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind == "binarize":
        return {"case": case, "x": _features(case, case["k0"], gen)}
    if kind == "expand":
        return {"case": case, "x": _features(case, case["raw"], gen), "seed": int(seed)}
    widths = (case["k0"],) + (case["k"],) * case["layers"]
    net = B.BMLP(widths, case["classes"], case["bound"], case["batch"], case["group"], R, int(seed))
    st = {"case": case, "net": net, "t": 0, "p_r": P_R}
    n = case["batch"]
    if kind in ("forward", "eval"):
        st["x"], st["y"] = _samples(case, net, n, gen)
        return st
    x, y = _samples(case, net, n * case["sets"], gen)
    layers = range(1, case["layers"] + 1)
    st["weights"] = {"h": [net.H_planes(l) for l in layers], "w": [net.W(l) for l in layers]}
    if kind == "epoch":
        st["x"], st["y"] = x, y
        st["orders"] = [torch.randperm(n * case["sets"], generator=gen, device=DEV, dtype=torch.int32) for _ in range(3)]
    else:
        st["x"], st["y"] = list(x.split(n)), list(y.split(n))
        st["stats"] = torch.empty((case["layers"], B.STATS_STRIDE), dtype=torch.int32, device=DEV)
    return st


def run(state):
    kind = state["case"]["kind"]
    if kind == "step":
        t = state["t"]
        i = t % len(state["x"])
        state["t"] = t + 1
        stats = state["net"].train_step(state["x"][i], state["y"][i], t, P_R, stats=state["stats"])
        return {"stats": stats, "weights": state["weights"]}
    if kind == "epoch":
        e, sets = state["t"], state["case"]["sets"]
        state["t"] = e + 1
        state["p_r"], err, stats = state["net"].train_epoch(state["x"], state["y"], state["orders"][e % 3], e * sets,
                                                            state["p_r"])
        return {"p_r": state["p_r"], "error": err, "stats": stats, "weights": state["weights"]}
    if kind == "forward":
        return state["net"].forward(state["x"])
    if kind == "eval":
        return state["net"].eval_exit(state["x"], state["y"])
    if kind == "binarize":
        median = B.feature_median(state["x"])
        return {"median": median, "bits": B.binarize(state["x"], median)}
    return B.expand(state["x"], state["case"]["k0"], state["seed"])


def work(case):
    n, kind = case["batch"], case["kind"]
    if kind == "binarize":
        return {"bytes": n * case["k0"] * 9 / 8, "flops": n * case["k0"]}
    if kind == "expand":
        return {"bytes": n * (case["raw"] + case["k0"] / 8), "flops": 2 * n * case["raw"] * case["k0"]}
    c, planes = case["classes"], case["bound"].bit_length()
    widths = [case["k0"]] + [case["k"]] * case["layers"]
    flops = bytes_ = 0
    for a, b in zip(widths, widths[1:]):
        flops += 2 * n * b * (a + c)
        bytes_ += b * a / 8 + c * b / 8
        if kind in ("step", "epoch"):      # hidden weights read and written, visible weights written
            bytes_ += (2 * planes + 1) * a * b / 8
        elif kind == "forward":
            bytes_ += 4 * n * c
    bytes_ += n * (case["k0"] / 8 + 4)
    steps = case["sets"] if kind == "epoch" else 1
    return {"bytes": steps * bytes_, "flops": steps * flops}


def tolerance(case):
    # Integer sums, counts, comparisons and counter-based draws: another correct implementation gives the same values.
    return "exact"


# The same results in plain torch, with every contraction in 64-bit floating point.


def _unpack(rows, k):
    """int64 bit rows -> ±1 in float64 [n][k]."""
    b = rows.contiguous().view(torch.uint8)
    bits = (b.unsqueeze(-1) >> torch.arange(8, device=DEV, dtype=torch.uint8)) & 1
    return bits.reshape(rows.shape[0], -1)[:, :k].double() * 2 - 1


def _bytes(bits, columns):
    """Boolean [n][k] -> uint8 [n][columns / 8], least significant bit first, zero past k."""
    pad = torch.zeros((bits.shape[0], columns), dtype=torch.uint8, device=DEV)
    pad[:, :bits.shape[1]] = bits
    weights = 2 ** torch.arange(8, device=DEV, dtype=torch.uint8)
    return (pad.view(bits.shape[0], -1, 8) * weights).sum(-1, dtype=torch.uint8)


def _words(bits):
    return _bytes(bits, (bits.shape[1] + 63) // 64 * 64).view(torch.int64)


def _philox(block, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors of 32-bit words."""
    def mul(a, m):
        low, high = (a & 0xFFFF) * m, (a >> 16) * m
        mid = high + (low >> 16)
        return mid >> 16, ((mid & 0xFFFF) << 16) | (low & 0xFFFF)
    full = torch.full_like
    c = [block & 0xFFFFFFFF, full(block, c1), full(block, c2), full(block, c3)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32 & 0xFFFFFFFF
    for _ in range(10):
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _bits_of(words, count):
    """The bits of int64 tensors of 32-bit words [..., m], in order, as [..., 32 m][:count]."""
    return ((words.unsqueeze(-1) >> torch.arange(32, device=DEV)) & 1).reshape(*words.shape[:-1], -1)[..., :count]


def _fired(k_out, k_in, layer, t, seed, threshold):
    """Which hidden weights reinforce: 32-bit draws (u8, u24) below the threshold."""
    groups = (k_in + 31) // 32
    q = torch.arange(k_out * groups, device=DEV).view(k_out, groups)
    u8 = torch.zeros((k_out, k_in), dtype=torch.int16, device=DEV)
    for half in (0, 1):
        for w, word in enumerate(_philox(2 * q + half, layer - 1, t, 3, seed)):
            u8 += _bits_of(word, k_in).to(torch.int16) << (4 * half + w)
    hi, lo = threshold >> 24, threshold & 0xFFFFFF
    fire = u8 < hi
    row, col = torch.nonzero(u8 == hi, as_tuple=True)
    j = row * k_in + col
    fine = torch.stack(_philox(j >> 2, layer - 1, t, 4, seed), -1).gather(-1, (j & 3).unsqueeze(-1)).squeeze(-1)
    fire[row, col] = (fine & 0xFFFFFF) < lo
    return fire


def _local(a, p):
    """Local outputs, first argmax, and the margin between the two largest."""
    y_hat = a @ p.t()
    c = y_hat.shape[1]
    pred = (y_hat * c - torch.arange(c, device=DEV)).argmax(1)
    top = y_hat.topk(2, 1).values
    return y_hat, pred, top[:, 0] - top[:, 1]


class _Exact:
    """A network's weights as float64 matrices, and its training step."""

    def __init__(self, case, net):
        self.seed, self.bound = int(net.cfg.seed), case["bound"]
        self.info = net.info
        layers = range(1, case["layers"] + 1)
        self.h = [net.H(l) for l in layers]
        self.p = [_unpack(net.P(l), case["k"]) for l in layers]

    def step(self, x, y, t, p_r):
        y, a, stats, new = y.long(), x, [], []
        for l, (h, p, i) in enumerate(zip(self.h, self.p, self.info), 1):
            z = a @ torch.where(h > 0, 1.0, -1.0).double().t()
            out = torch.where(z >= 0, 1.0, -1.0).double()
            _, pred, tau = _local(out, p)
            err = pred != y
            upd = err | (tau < math.ceil(R * i.k_out))
            rho = p[y]
            key = torch.where(z * rho < 0, z.abs() * i.k_out + torch.arange(i.k_out, device=DEV), math.inf)
            best, at = key.view(len(y), i.groups, i.gamma).min(-1)
            pick = (at + torch.arange(i.groups, device=DEV) * i.gamma)[best.isfinite() & upd[:, None]]
            mu = torch.nonzero(best.isfinite() & upd[:, None])[:, 0]
            sel = torch.zeros_like(rho)
            sel[mu, pick] = rho[mu, pick]
            fired = 0
            if upd.any():
                h = (h.double() + 2 * (sel.t() @ a)).clamp_(-self.bound, self.bound)
                q = p_r * math.sqrt(2.0 / (math.pi * i.k_out))
                fire = _fired(i.k_out, i.k_in, l, t, self.seed, min(2 ** 32, math.ceil(q * 2 ** 32)))
                fired = int(fire.sum())
                h = (h + 2 * fire * torch.sign(h)).clamp_(-self.bound, self.bound).to(torch.int8)
            new.append(h)
            stats.append([int(err.sum()), int(upd.sum()), len(mu), fired])
            a = out
        self.h = new
        return torch.tensor(stats, dtype=torch.int32)

    def weights(self):
        planes = []
        for h, i in zip(self.h, self.info):
            u = (h.to(torch.int16) + self.bound) // 2
            planes.append(torch.cat([_bytes((u >> q) & 1, 32 * i.h_ps) for q in range(i.h_planes)], 1))
        return {"h": planes, "w": [_words(h > 0) for h in self.h]}


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    if kind == "binarize":
        x = st["x"]
        median = x.double().sort(0).values[(len(x) - 1) // 2].to(torch.int8)
        return {"median": median, "bits": _words(x >= median)}
    if kind == "expand":
        raw, k0 = case["raw"], case["k0"]
        blocks = torch.arange((k0 * raw + 127) // 128, device=DEV)
        r = _bits_of(torch.stack(_philox(blocks, 0xFFFFFFFF, 0, 5, st["seed"]), -1), 128).reshape(-1)[:k0 * raw]
        return _words(st["x"].double() @ (r.view(k0, raw).double() * 2 - 1).t() >= 0)
    net = _Exact(case, st["net"])
    if kind == "step":
        stats = net.step(_unpack(st["x"][0], case["k0"]), st["y"][0], 0, P_R)
        return {"stats": stats, "weights": net.weights()}
    if kind == "epoch":
        n, wrong, stats = case["batch"], 0, []
        for b in range(case["sets"]):
            at = st["orders"][0][b * n:(b + 1) * n].long()
            stats.append(net.step(_unpack(st["x"][at], case["k0"]), st["y"][at], b, P_R))
            wrong += int(stats[-1][-1, 0])
        error = wrong / (n * case["sets"])
        return {"p_r": P_R * math.sqrt(error), "error": error, "stats": torch.stack(stats), "weights": net.weights()}
    a, outs, left = _unpack(st["x"], case["k0"]), [], torch.ones(case["batch"], dtype=torch.bool, device=DEV)
    for l, (h, p) in enumerate(zip(net.h, net.p), 1):
        a = torch.where(a @ torch.where(h > 0, 1.0, -1.0).double().t() >= 0, 1.0, -1.0).double()
        y_hat, pred, tau = _local(a, p)
        if kind == "forward":
            outs.append(y_hat.to(torch.int32))
            continue
        ok = pred == st["y"]
        leave = left & ((tau >= math.ceil(R * case["k"])) | (l == case["layers"]))
        left = left & ~leave
        outs.append(torch.stack([ok.sum(), leave.sum(), (ok & leave).sum()]).to(torch.int32))
    return torch.stack(outs)
