"""Whole passes in which the choices that depend on a layer's size fall the other way than on the small nets: layers
of at least 2 GFLOP run through the tile transforms in a training or inference pass, and inference makes the weights'
other forms on a side stream.  Every test checks from the names of the launched kernels which way each stage went."""
import numpy as np
import pytest
import torch

import synthetic_inputs as S
from gpu_common import TENSOR_RTOL, build_pair, cuda, run_step_and_compare
from helpers import rel_l2
from oracle import alexnet_oracle as O

pytestmark = pytest.mark.gpu

# 3x3 and 5x5 unit-stride layers with paddings 0, 1 and 2, one and two groups and channel counts that fill no tile, each
# above 2 GFLOP at a batch of 32: 67 -> pool 33 -> 33 -> 31 -> 33 -> 33 (pool 16)
WIDE = {
    "name": "wide", "in_c": 3, "crop": 67, "raw": 67,
    "conv": [(48, 3, 1, 1, 1, 1, 1), (56, 5, 1, 2, 2, 0, 0), (76, 3, 1, 0, 1, 0, 0), (80, 3, 1, 2, 1, 0, 0),
             (88, 3, 1, 1, 2, 0, 1)],
    "fc": [40, 24, 5], "lrn": (5, 2.0, 1e-4, 0.75), "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9, "weight_decay": 5e-4,
}
# 4x4 maps, one 4x4 tile per picture, 2.03 GFLOP a layer at a batch of 64
ONE_TILE = dict(WIDE, name="one_tile", crop=9, raw=9,
                conv=[(332, 3, 2, 0, 1, 0, 0)] + [(332, 3, 1, 1, 1, 0, 0)] * 4, fc=[8, 8, 4])


def kernels_of(lib, run):
    """The names of the kernels that run() launches, with the layer and pass they belong to, and its result."""
    lib.profile_begin()
    try:
        out = run()
        torch.cuda.synchronize()
    finally:
        entries = lib.profile_end(1024)
    return {e["name"] for e in entries}, out


def transformed(names, what):
    """Numbers of the convolution stages whose pass `what` (fwd, bwd_w, bwd_x) ran through the tile transforms."""
    kernel = {"fwd": "wino_in", "bwd_w": "wino_dy", "bwd_x": "wino_dx"}[what]
    return [i for i in range(1, 6) if f"conv{i}.{what}:{kernel}" in names]


@pytest.mark.parametrize("wl,batch,std", [(WIDE, 32, 0.05), (ONE_TILE, 64, 0.02)], ids=["wide", "one_tile"])
def test_steps_with_transformed_stages(lib, wl, batch, std):
    """Two steps against the oracle; parameters are updated at the end of each, taps transformed in line."""
    names, _ = kernels_of(lib, lambda: run_step_and_compare(lib, wl, batch, seed=14, bias=0.05, std=std, use_raw=False,
                                                            steps=2, mom_std=0.01, direct=False))
    for what in ("fwd", "bwd_w", "bwd_x"):
        assert transformed(names, what) == [2, 3, 4, 5], what


def test_train_step_with_transformed_stages_equals_its_parts(lib):
    """train_step transforms the taps on the side stream and updates the dense layers early; the same bits."""
    batch, classes = 32, WIDE["fc"][-1]
    a, _, _, _ = build_pair(lib, WIDE, batch, seed=4, pseed=4, std=0.05, bias=0.1)
    b, _, _, _ = build_pair(lib, WIDE, batch, seed=4, pseed=4, std=0.05, bias=0.1)
    for step in range(3):
        x, labels = S.make_float_batch(batch, 3, 67, 67, classes, 40 + step)
        for net in (a, b):
            net.set_input(cuda(x), step % 2)
        names, la = kernels_of(lib, lambda: float(a.train_step(cuda(labels), step, slot=step % 2).cpu().item()))
        assert transformed(names, "bwd_x") == [2, 3, 4, 5]
        lb = float(b.forward_backward(cuda(labels), step, slot=step % 2).cpu().item())
        b.apply_update()
        assert la == lb, (step, la, lb)
    pa, pb, ma, mb = a.get_params(), b.get_params(), a.get_momentum(), b.get_momentum()
    for k in pa:
        assert np.array_equal(pa[k], pb[k]) and np.array_equal(ma[k], mb[k]), k
    a.close()
    b.close()


@pytest.mark.timeout(300)
def test_step_with_some_stages_transformed_and_others_direct(lib):
    """The full net at a batch of 8: conv2 and conv3 are above the line, conv4 (1.8 GFLOP) and conv5 (1.2) below."""
    names, _ = kernels_of(lib, lambda: run_step_and_compare(lib, S.ALEXNET, 8, seed=18, bias=0.1, std=0.02, use_raw=False,
                                                            mom_std=0.001, direct=False))
    for what in ("fwd", "bwd_w", "bwd_x"):
        assert transformed(names, what) == [2, 3], what


@pytest.mark.parametrize("wl,batch,precision,paired", [(S.MINI, 16, 0, True), (S.MINI, 16, 1, True), (S.ALEXNET, 8, 0, False),
                                                       (S.ALEXNET, 8, 1, False)])
def test_profile_names_every_gradient(lib, wl, batch, precision, paired):
    """A product's time is found under its layer and pass: both gradients under .bwd where they are one launch, else each under
    its own name."""
    net = lib.AlexNet(wl, batch, precision=precision)
    x, labels = S.make_float_batch(batch, wl["in_c"], wl["crop"], wl["crop"], wl["fc"][-1], 3)
    net.set_input(cuda(x), 0)
    names, _ = kernels_of(lib, lambda: net.forward_backward(cuda(labels), 0))
    products = {n.split(":")[0] for n in names if n.split(":")[-1].startswith("gemm")}
    for layer in ("fc6", "fc7", "fc8", "conv2"):
        want = {layer + ".fwd"} | ({layer + ".bwd"} if paired else {layer + ".bwd_w", layer + ".bwd_x"})
        assert {p for p in products if p.startswith(layer + ".")} == want
    assert "conv1.bwd_w" in products
    net.close()


# ------------------------------------------------------------- inference ---
def spread_params(net, seed):
    """Weights N(0, 1/fan_in) and small biases: logits of order one."""
    rng = np.random.default_rng(seed)
    return {k: (rng.standard_normal(s) / np.sqrt(np.prod(s[1:])) if k.endswith(".w") else rng.standard_normal(s) * 0.1)
            .astype(np.float32) for k, s in net.shapes.items()}


# precision, batch, stages transformed, forked onto the side stream, dense weights copied to bf16
@pytest.mark.timeout(300)
@pytest.mark.parametrize("precision,batch,stages,fork,copy", [
    (0, 6, [2], True, False),              # one stage transformed, the others direct
    (0, 16, [2, 3, 4, 5], True, False),
    (1, 4, [], False, False),              # dense layers on a few rows read the fp32 weights
    (1, 16, [], False, True),              # copies made in line
    (1, 80, [], True, True),               # copies made on the side stream under the first layer
])
def test_inference_uses_the_parameters_of_the_call(lib, precision, batch, stages, fork, copy):
    """Two calls on one handle with other parameters and pictures in between: each returns the bits that a handle which
    has seen nothing else returns, and so does the validation pass, whose counts follow from the same logits."""
    wl = S.ALEXNET
    net = lib.AlexNet(wl, batch, precision=precision)
    sets = [spread_params(net, 1), spread_params(net, 2)]
    xs = [S.make_float_batch(batch, 3, 227, 227, 1000, 60 + i) for i in range(2)]
    flat = [cuda(net.flatten(p)) for p in sets]
    pictures = [cuda(x) for x, _ in xs]
    got = []
    for p, x in zip(flat, pictures):  # nothing waits between the calls but the copies of the parameters
        net.set_params(p)
        names, probs = kernels_of(lib, lambda: net.forward(x))
        assert transformed(names, "fwd") == stages
        assert ("fc.weights16:to_bf16" in names) == (fork and copy)
        assert any(n.endswith(":to_bf16") and n.startswith("fc.") or n == "to_bf16" for n in names) == copy
        assert any("fc_rows" in n for n in names) == (batch <= 4)
        got.append((probs.cpu().numpy(), net.tensor(lib.T_FC_ACT, 8)))
    labels = got[1][1].reshape(batch, -1).argsort(1)[np.arange(batch), -1 - np.arange(batch) % 8].astype(np.int32)
    counts = torch.zeros(3, dtype=torch.int32, device="cuda")
    net.set_input(pictures[0], 0)
    net.set_input(pictures[1], 1)
    net.validate(cuda(labels), [1, 3, 5], counts, slot=1)
    assert np.array_equal(net.tensor(lib.T_FC_ACT, 8), got[1][1])
    assert counts.cpu().tolist() == [int((np.arange(batch) % 8 < k).sum()) for k in (1, 3, 5)]
    net.close()
    for p, x, (probs, logits) in zip(flat, pictures, got):
        fresh = lib.AlexNet(wl, batch, precision=precision)
        fresh.set_params(p)
        assert np.array_equal(fresh.forward(x).cpu().numpy(), probs)
        fresh.close()
        ref = lib.AlexNet(wl, batch, flags=lib.FLAG_DIRECT_CONV)  # no transforms, no copies
        ref.set_params(p)
        assert rel_l2(probs, ref.forward(x).cpu().numpy()) <= (2e-2 if precision else 1e-5)
        ref.close()
    assert rel_l2(got[0][0], got[1][0]) > 0.1


@pytest.mark.timeout(300)
def test_inference_of_the_full_net_against_the_oracle(lib):
    """One stage transformed, the others direct, on the caller's pictures."""
    batch = 6
    net, spec, _, _ = build_pair(lib, S.ALEXNET, batch, seed=3)
    p32 = spread_params(net, 5)
    net.set_params(p32)
    x, _ = S.make_float_batch(batch, 3, 227, 227, 1000, 70)
    want = O.forward(spec, {k: v.astype(np.float64) for k, v in p32.items()}, x.astype(np.float64))
    assert rel_l2(net.forward(cuda(x)).cpu().numpy(), want) <= TENSOR_RTOL
    net.close()


@pytest.mark.parametrize("wl,batch,precision", [(S.MIDI, 5, 0), (S.ALEXNET, 6, 0), (S.ALEXNET, 80, 1)],
                         ids=["no_fork", "fp32", "bf16"])
def test_inference_in_a_captured_graph(lib, wl, batch, precision):
    """The fork onto the side stream joins in the same call: a graph captured from it is replayed with other pictures and
    other parameters, with eager passes in between."""
    net = lib.AlexNet(wl, batch, precision=precision)
    size, classes = wl["crop"], wl["fc"][-1]
    x = cuda(S.make_float_batch(batch, 3, size, size, classes, 80)[0])
    net.set_params(spread_params(net, 7))
    net.forward(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        probs = net.forward(x)
    for i in range(4):
        x.copy_(cuda(S.make_float_batch(batch, 3, size, size, classes, 81 + i)[0]))
        net.set_params(spread_params(net, 8 + i))
        graph.replay()
        torch.cuda.synchronize()
        got = probs.cpu().numpy()
        assert np.array_equal(got, net.forward(x).cpu().numpy()), i
    net.close()
