"""Timed workloads of the AlexNet training and inference path.

A case is one call sequence of a user's program on one MI355X: a training
iteration from stored pictures (preprocess, forward, backward, update), an
inference pass on a preprocessed batch, or an iteration of two replicas that
exchange and average.  Networks are the tables of synthetic_inputs.py; batch
sizes run from one picture to 256, the largest configuration of bench.py.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

import synthetic_inputs as S
from paper_1412_2302_amd import binding as B

PRECISION = {"fp32": 0, "bf16": 1}


def listed():
    return [
        # smallest iterations: a few MFLOP per launch, so launches and latency are what they cost
        dict(name="train_mini_b16_fp32", kind="train", net="mini", batch=16, precision="fp32"),
        dict(name="train_mini_b128_bf16", kind="train", net="mini", batch=128, precision="bf16"),
        # channel counts 24/40/72 and dense widths 200/136/37: no dimension is a multiple of a tile
        dict(name="train_midi_b48_fp32", kind="train", net="midi", batch=48, precision="fp32"),
        # serving one picture: bound by reading the weights once
        dict(name="infer_b1_fp32", kind="infer", net="alexnet", batch=1, precision="fp32"),
        # serving a batch that fills no tile
        dict(name="infer_b50_fp32", kind="infer", net="alexnet", batch=50, precision="fp32"),
        # validation pass over a large batch with reduced-precision products
        dict(name="infer_b256_bf16", kind="infer", net="alexnet", batch=256, precision="bf16"),
        # last, ragged minibatch of an epoch
        dict(name="train_b37_fp32", kind="train", net="alexnet", batch=37, precision="fp32"),
        # the per-replica minibatch of the paper
        dict(name="train_b128_fp32", kind="train", net="alexnet", batch=128, precision="fp32"),
        # the paper's single-GPU batch, both precisions
        dict(name="train_b256_fp32", kind="train", net="alexnet", batch=256, precision="fp32"),
        dict(name="train_b256_bf16", kind="train", net="alexnet", batch=256, precision="bf16"),
        # a small per-replica minibatch with reduced-precision products
        dict(name="train_b64_bf16", kind="train", net="alexnet", batch=64, precision="bf16"),
        # two replicas on one GPU, weights and momentum averaged after the step
        dict(name="replicas_b64_fp32", kind="replicas", net="alexnet", batch=64, precision="fp32"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Inference from one picture up, training from the smallest minibatch in earnest use up; never a listed case."""
    taken = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    while True:
        kind = rng.choice(["train", "train", "train", "infer", "infer", "replicas"])
        net = rng.choice(["alexnet"] * 4 + ["mini", "midi"])
        lo, hi = (1, 256) if kind == "infer" else (16, 256) if kind == "train" else (16, 96)
        case = dict(kind=kind, net=net, batch=_log_int(rng, lo, hi), precision=rng.choice(["fp32", "fp32", "bf16"]))
        if case not in taken:
            return case


# ------------------------------------------------------------------ inputs ---
def _pictures(gen, batch, c, size):
    """Stored uint8 pictures: smooth regions with fine detail on top, as photographs have."""
    coarse = torch.rand((batch, c, 9, 9), generator=gen, device="cuda") * 200.0 + 20.0
    x = F.interpolate(coarse, size=(size, size), mode="bilinear", align_corners=True)
    x += torch.randn(x.shape, generator=gen, device="cuda") * 20.0
    return x.clamp_(0, 255).to(torch.uint8)


def _weights(gen, net, scale):
    """Canonical flat vector with weights N(0, scale^2 / fan_in) and zero biases."""
    parts = []
    for name, shape in net.shapes.items():
        n = math.prod(shape)
        if name.endswith(".b"):
            parts.append(torch.zeros(n, device="cuda"))
        else:
            parts.append(torch.randn(n, generator=gen, device="cuda") * (scale / math.sqrt(math.prod(shape[1:]))))
    return torch.cat(parts)


def _handle(case, seed):
    return B.AlexNet(S.WORKLOADS[case["net"]], case["batch"], seed=seed, precision=PRECISION[case["precision"]])


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    wl, batch = S.WORKLOADS[case["net"]], case["batch"]
    net = _handle(case, seed)
    # a network that serves has spread logits; one in early training has nearly even ones
    params = _weights(gen, net, 1.0 if case["kind"] == "infer" else 0.7)
    net.set_params(params)
    if case["kind"] == "infer":
        return {"kind": "infer", "net": net, "x": _pictures(gen, batch, wl["in_c"], wl["crop"]).float() - 120.0}
    momentum = _weights(gen, net, 0.01)  # training under way: updates of about 1 % of the weights
    replicas = [net]
    net.set_momentum(momentum)
    if case["kind"] == "replicas":  # created identically, fed different pictures
        replicas.append(_handle(case, seed + 1))
        replicas[1].set_params(params)
        replicas[1].set_momentum(momentum)
    fed = [(r, _pictures(gen, batch, wl["in_c"], wl["raw"]),
            torch.randint(0, wl["fc"][-1], (batch,), generator=gen, device="cuda", dtype=torch.int32))
           for r in replicas]
    mean = torch.rand((wl["in_c"], wl["raw"], wl["raw"]), generator=gen, device="cuda") * 40.0 + 100.0
    return {"kind": case["kind"], "step": 0, "mean": mean, "nets": fed}


# --------------------------------------------------------------------- run ---
def run(state):
    if state["kind"] == "infer":
        return state["net"].forward(state["x"])
    step = state["step"]
    state["step"] += 1
    for net, raw, labels in state["nets"]:
        net.preprocess(raw, state["mean"], step, step % 2)
        net.train_step(labels, step, slot=step % 2)
    if state["kind"] == "replicas":
        B.average_replicas(state["nets"][0][0], state["nets"][1][0])
    return [{"loss": net.loss, "params": net.params, "momentum": net.momentum} for net, _, _ in state["nets"]]


# -------------------------------------------------------------------- work ---
def _layers(wl):
    """(multiply-adds per picture, weights) of every layer, and whether its data gradient is needed."""
    c, h = wl["in_c"], wl["crop"]
    out = []
    for i, (co, k, st, pd, g, _lrn, pool) in enumerate(wl["conv"]):
        h = (h + 2 * pd - k) // st + 1
        w = co * (c // g) * k * k
        out.append((h * h * w, w + co, i > 0))
        h = (h - 3) // 2 + 1 if pool else h
        c = co
    fin = c * h * h
    for f in wl["fc"]:
        out.append((fin * f, fin * f + f, True))
        fin = f
    return out


def work(case):
    """Multiply-adds by the definition of every layer; weights (and momentum) and pictures once, results once."""
    wl, b = S.WORKLOADS[case["net"]], case["batch"]
    layers = _layers(wl)
    n_params = sum(p for _, p, _ in layers)
    if case["kind"] == "infer":
        pixels = wl["in_c"] * wl["crop"] ** 2
        return {"bytes": 4.0 * (n_params + b * pixels + b * wl["fc"][-1]), "flops": 2.0 * b * sum(m for m, _, _ in layers)}
    replicas = 2 if case["kind"] == "replicas" else 1
    pixels = wl["in_c"] * wl["raw"] ** 2
    flops = 2.0 * b * sum(m * (3 if dx else 2) for m, _, dx in layers)
    return {"bytes": replicas * (16.0 * n_params + b * pixels + 4.0 * b), "flops": replicas * flops}


def tolerance(case):
    """About four times what one pass differs by between the direct and the tile-transformed convolutions, with
    and without split reductions (the same sums in other orders), over two steps on one state.

    A training step contains ReLU gates and pooling winners, and a few of its 1e8 units lie within rounding of a
    change: each one that falls the other way moves single gradients, so momentum differs by far more than the sums
    themselves do (1e-6), and with bf16 products, whose stored activations round to 8 bits, by 4e-2 of the gradient;
    a gradient is 2 to 10 % of the momentum here and falls with the square root of the batch."""
    bf16 = case["precision"] == "bf16"
    if case["kind"] == "infer":
        return {"rel": 6e-3, "max": 4e-2} if bf16 else {"rel": 6e-6, "max": 3e-5}
    if bf16:
        return {"rel": min(0.03, 0.12 / math.sqrt(case["batch"])), "max": 0.99}
    return {"rel": 2.5e-3, "max": 0.6}

# ------------------------------------------------------------------- exact ---
def _shapes(wl):
    """(name, shape) of every parameter in the order of the flat vector: all weights, then all biases."""
    weights, c, h = [], wl["in_c"], wl["crop"]
    for i, (co, k, st, pd, g, _lrn, pool) in enumerate(wl["conv"]):
        weights.append(("conv%d" % (i + 1), (co, c // g, k, k)))
        h = (h + 2 * pd - k) // st + 1
        h = (h - 3) // 2 + 1 if pool else h
        c = co
    fin = c * h * h
    for j, f in enumerate(wl["fc"]):
        weights.append(("fc%d" % (len(wl["conv"]) + 1 + j), (f, fin)))
        fin = f
    return {**{n + ".w": s for n, s in weights}, **{n + ".b": s[:1] for n, s in weights}}


class _Table:
    def __init__(self, wl):
        self.shapes = _shapes(wl)


def _logits64(wl, flat, x, masks):
    """Logits in 64 bits; masks: dropout masks while training, None for inference (activations scaled by 1 - p)."""
    p, at = {}, 0
    for name, shape in _shapes(wl).items():
        n = math.prod(shape)
        p[name], at = flat[at:at + n].double().view(shape), at + n
    lrn_n, lrn_k, alpha, beta = wl["lrn"]
    rows = []
    for h in x.split(32):  # the unfolded pictures of 32 stay below 1 GB
        for i, (co, k, st, pd, g, lrn, pool) in enumerate(wl["conv"]):
            w, b = p["conv%d.w" % (i + 1)], p["conv%d.b" % (i + 1)]
            side = (h.shape[2] + 2 * pd - k) // st + 1
            parts = [torch.matmul(wg.reshape(co // g, -1), F.unfold(hg, k, padding=pd, stride=st))
                     for wg, hg in zip(w.chunk(g), h.chunk(g, 1))]
            h = F.relu(torch.cat(parts, 1).view(h.shape[0], co, side, side) + b.view(1, -1, 1, 1))
            if lrn:
                sq = F.pad(h * h, (0, 0, 0, 0, lrn_n // 2, lrn_n // 2))
                s = lrn_k + alpha * sum(sq[:, d:d + co] for d in range(lrn_n))
                h = h * s ** -beta
            if pool:
                h = h.unfold(2, 3, 2).unfold(3, 3, 2).amax((-1, -2))
        rows.append(h.flatten(1))
    h = torch.cat(rows)
    first = len(wl["conv"]) + 1
    for j in range(len(wl["fc"])):
        h = h @ p["fc%d.w" % (first + j)].t() + p["fc%d.b" % (first + j)]
        if j + 1 < len(wl["fc"]):
            h = F.relu(h) * (masks[j] if masks else 1.0 - wl["dropout_p"])
    return h


def _hash(seed, step, tag, count):
    """The counter-based generator of crops, mirrors and dropout: splitmix64 of (seed, step, purpose, index)."""
    z = np.array([seed + 0x9E3779B97F4A7C15 & 0xFFFFFFFFFFFFFFFF], np.uint64)

    def mix(v):
        v = (v ^ v >> np.uint64(30)) * np.uint64(0xBF58476D1CE4E5B9)
        v = (v ^ v >> np.uint64(27)) * np.uint64(0x94D049BB133111EB)
        return v ^ v >> np.uint64(31)
    key = mix(mix(z) ^ np.uint64(step))
    return mix(key ^ np.uint64(tag << 56) ^ np.arange(count, dtype=np.uint64))


def _loss64(wl, seed, params, raw, labels, mean):
    """Mean cross-entropy of step 0 in 64 bits: crop and mirror, forward with dropout."""
    batch, crop, room = raw.shape[0], wl["crop"], np.uint64(wl["raw"] - wl["crop"] + 1)
    ox, oy = (((_hash(seed, 0, t, batch) >> np.uint64(32)) % room).astype(int) for t in (1, 2))
    flip = (_hash(seed, 0, 3, batch) >> np.uint64(63)).astype(bool)
    x = torch.stack([(raw[i].double() - mean.double())[:, oy[i]:oy[i] + crop, ox[i]:ox[i] + crop].flip((2,) if flip[i] else ())
                     for i in range(batch)])
    thresh = np.uint64(int(wl["dropout_p"] * (1 << 24)))
    masks = [torch.from_numpy((_hash(seed, 0, tag, batch * f) >> np.uint64(40)) >= thresh).view(batch, f).cuda().double()
             for tag, f in zip((6, 7), wl["fc"])]
    return F.cross_entropy(_logits64(wl, params, x, masks), labels.long()).view(1)


def exact(case, seed):
    """Probabilities and losses in 64 bits.  Updated weights and momentum have no such value: a training step's
    gradient depends on which side of zero each ReLU input and which tap of each pooling window is taken as the
    larger, and a few of the 1e8 choices lie within rounding (see tolerance()).  With bf16 products the mean loss has
    none worth comparing either: the pictures' errors have either sign and what is left of their sum is chance."""
    if case["kind"] != "infer" and case["precision"] == "bf16":
        return None
    gen = torch.Generator(device="cuda").manual_seed(seed)
    wl, batch = S.WORKLOADS[case["net"]], case["batch"]
    params = _weights(gen, _Table(wl), 1.0 if case["kind"] == "infer" else 0.7)
    if case["kind"] == "infer":
        x = _pictures(gen, batch, wl["in_c"], wl["crop"]).float() - 120.0
        return _logits64(wl, params, x.double(), None).softmax(1)
    _weights(gen, _Table(wl), 0.01)
    out, seeds = [], [seed, seed + 1] if case["kind"] == "replicas" else [seed]
    fed = [(s, _pictures(gen, batch, wl["in_c"], wl["raw"]),
            torch.randint(0, wl["fc"][-1], (batch,), generator=gen, device="cuda", dtype=torch.int32)) for s in seeds]
    mean = torch.rand((wl["in_c"], wl["raw"], wl["raw"]), generator=gen, device="cuda") * 40.0 + 100.0
    for s, raw, labels in fed:
        out.append({"loss": _loss64(wl, s, params, raw, labels, mean), "params": None, "momentum": None})
    return out
