"""Whole training steps of bf16 handles, every product against 64 bits of its own operands: activations and gradients are read
back, rounded to bf16 as the products have them, and multiplied in double precision.  So each product of a pass is held to
what its fp32 sums round, whichever kernel took it -- among them stages whose weight gradient alone is a small product, and
dense layers over operands stored as bf16, which no operator of their own reaches."""
import numpy as np
import pytest
import torch

import synthetic_inputs as S
from gpu_common import cuda
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def bf(a, rounded=True):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.bfloat16() if rounded else t).double()


def with_dense(wl, widths, last_pool=None):
    wl = dict(wl, fc=widths)
    if last_pool is not None:
        wl["conv"] = [*wl["conv"][:-1], (*wl["conv"][-1][:-1], last_pool)]
    return wl


# Sums of products that are exact in fp32: of n terms with independent rounding sqrt(n/2) * 2^-24 of the result, 5e-6 at the
# 14000 that the longest slice has here.  A gradient that is rounded to bf16 once more on the way (dense layers below the
# last) lies the other way where 64 bits and fp32 sums fall on two sides of a rounding boundary: about 1e-6 / 2^-8 of the
# elements by 2^-8 each, sqrt(2.6e-4) * 2^-8 = 6e-5.
SUMS, ROUNDED = 5e-6, 1e-4


@pytest.mark.parametrize("wl,batch", [
    (S.PADS, 290),  # second stage: 64 slices of a direct weight gradient where a small product would have 148
    (S.PADS, 33), (S.MINI, 60), (S.MINI, 240), (S.MINI, 400), (S.MIDI, 40), (S.ALEXNET, 8),
    (with_dense(S.MINI, [2056, 1032, 504], 0), 70), (with_dense(S.MINI, [2056, 1032, 504], 0), 37),
    (with_dense(S.MINI, [4104, 2056, 200], 0), 130), (with_dense(S.MINI, [264, 1040, 1000], 0), 17)])
def test_every_product_of_a_step(lib, wl, batch):
    wl = dict(wl, dropout_p=0.0, lr=0.0, momentum=0.0)  # the step's weights are the ones read back, no mask on the way
    net = lib.AlexNet(wl, batch, seed=3, precision=1)
    rng = np.random.default_rng(batch)
    params = {k: (rng.standard_normal(s) * (1.0 / np.sqrt(np.prod(s[1:])))).astype(np.float32) if k.endswith(".w") else
              (rng.standard_normal(s) * 0.1).astype(np.float32) for k, s in net.shapes.items()}
    net.set_params(params)
    x, labels = S.make_float_batch(batch, wl["in_c"], wl["crop"], wl["crop"], wl["fc"][-1], 11)
    net.set_input(cuda(x), 0)
    net.train_step(cuda(labels), 0, slot=0)
    net.check()
    g = net.get_grads()

    def close(name, got, want, tol=SUMS):
        want = want.numpy()
        got = np.asarray(got, np.float64).reshape(want.shape)
        assert rel_l2(got, want) <= tol, (name, rel_l2(got, want))
        worst = np.abs(got - want).max() / np.abs(want).max()  # no single wrong element
        assert worst <= max(1e-4, 2.0 ** -7 if tol > SUMS else 0.0), (name, worst)

    # ---- convolutions ----
    h, hi, gate = x, wl["crop"], None
    for i, (cout, k, st, pad, groups, lrn, pool) in enumerate(wl["conv"]):
        n, ho = "conv%d" % (i + 1), (hi + 2 * pad - k) // st + 1
        w, b = bf(params[n + ".w"]), torch.from_numpy(params[n + ".b"]).double()
        act = net.tensor(lib.T_CONV_ACT, i + 1).reshape(batch, cout, ho, ho)
        dact = net.tensor(lib.T_CONV_DACT, i + 1).reshape(batch, cout, ho, ho)
        close(n + " forward", act, torch.nn.functional.conv2d(bf(h), w, b, st, pad, 1, groups).relu())
        close(n + " weight gradient", g[n + ".w"],
              torch.nn.grad.conv2d_weight(bf(h), w.shape, bf(dact), st, pad, 1, groups))
        close(n + " bias gradient", g[n + ".b"], torch.from_numpy(dact).double().sum((0, 2, 3)))
        if gate is not None:  # the stage below takes this data gradient as its output gradient, through its ReLU
            want = torch.nn.grad.conv2d_input(tuple(h.shape), w, bf(dact), st, pad, 1, groups)
            close(n + " data gradient", below, want * (torch.from_numpy(gate) > 0))
        gate, below = (act, dact) if not lrn and not pool else (None, None)
        hi = (ho - 3) // 2 + 1 if pool else ho
        h = net.tensor(lib.T_POOL, i + 1).reshape(batch, cout, hi, hi) if pool else act
    # ---- dense layers; operands whose rows are no multiple of four floats stay in fp32 ----
    acts = [h.reshape(batch, -1)]
    for j in (6, 7, 8):
        n, fours = "fc%d" % j, acts[-1].shape[1] % 4 == 0
        y = net.tensor(lib.T_FC_ACT, j).reshape(batch, -1)
        want = bf(acts[-1], fours) @ bf(params[n + ".w"], fours).T + torch.from_numpy(params[n + ".b"]).double()
        close(n + " forward", y, want if j == 8 else want.relu())
        acts.append(y)
    dz = torch.from_numpy(net.tensor(lib.T_DLOGITS, 0).reshape(batch, -1)).double()
    for j in (8, 7, 6):
        n, a, tol = "fc%d" % j, acts[j - 6], SUMS if j == 8 else ROUNDED
        fours = a.shape[1] % 4 == 0 and dz.shape[1] % 4 == 0
        dz32 = dz.float().numpy()
        close(n + " weight gradient", g[n + ".w"], bf(dz32, fours).T @ bf(a, fours), tol)
        close(n + " bias gradient", g[n + ".b"], dz.sum(0), tol)
        dz = bf(dz32, fours) @ bf(params[n + ".w"], fours)
        if j > 6 or gate is not None:
            dz = dz * (torch.from_numpy(a if j > 6 else gate.reshape(batch, -1)) > 0)
    if gate is not None:
        close("fc6 data gradient", below, dz.reshape(below.shape), ROUNDED)
    net.close()
