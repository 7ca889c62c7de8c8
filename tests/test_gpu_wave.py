"""Small products (csrc/gemm_wave.h): layers whose sizes fill no 32 x 32 tile, no 16-deep step and no whole wave, through
the convolution operators of small nets, both precisions, and through whole training steps against the oracle."""
import numpy as np
import pytest
import torch

import synthetic_inputs as S
from gpu_common import cuda, run_step_and_compare
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def net_of(conv, crop, fc, in_c=3):
    return {"name": "edge", "in_c": in_c, "crop": crop, "raw": crop, "conv": conv, "fc": fc, "lrn": (5, 2.0, 1e-4, 0.75),
            "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9, "weight_decay": 5e-4}


# kernels of 1 to 15, strides, paddings past the map's edge, one to three groups, channels that are no multiple of anything,
# one pixel a map; a run-mode first layer (3 channels, no padding), a padded one and one of a single channel
NETS = {
    "odd_channels": net_of([(12, 7, 2, 0, 1, 0, 1), (20, 5, 1, 2, 2, 0, 0), (36, 3, 1, 1, 1, 0, 0), (44, 3, 1, 2, 4, 0, 0),
                            (28, 3, 1, 0, 2, 0, 1)], 37, [33, 18, 9]),
    "large_kernel": net_of([(8, 15, 1, 7, 1, 0, 0), (16, 15, 1, 7, 2, 0, 1), (8, 3, 1, 3, 1, 0, 0), (8, 1, 1, 0, 1, 0, 0),
                            (4, 2, 1, 0, 1, 0, 0)], 17, [16, 8, 8]),
    "one_pixel": net_of([(32, 3, 2, 1, 1, 0, 1), (32, 3, 1, 1, 1, 0, 0), (64, 3, 1, 1, 2, 0, 0), (33, 3, 1, 1, 1, 0, 0),
                         (8, 3, 1, 1, 1, 0, 0)], 6, [40, 12, 16], in_c=4),
    "one_channel": net_of([(4, 3, 1, 0, 1, 0, 1), (4, 3, 1, 1, 1, 0, 0), (8, 3, 1, 1, 1, 0, 0), (4, 3, 1, 1, 1, 0, 0),
                           (4, 3, 1, 1, 1, 0, 1)], 20, [9, 11, 10], in_c=1),
}


def reference(x, w, b, dy, geom):
    k, st, pd, g = geom
    x, w, b, dy = (torch.from_numpy(a).double() for a in (x, w, b, dy))
    x.requires_grad_(True)
    w.requires_grad_(True)
    y = torch.nn.functional.conv2d(x, w, b, stride=st, padding=pd, groups=g)
    y.backward(dy)
    return y.detach().numpy(), x.grad.numpy(), w.grad.numpy()


@pytest.mark.parametrize("name", NETS)
@pytest.mark.parametrize("batch", [1, 3, 17])
@pytest.mark.parametrize("precision", [0, 1])
def test_convolutions_at_the_edges(lib, name, batch, precision):
    """Every layer's three products.  fp32: a few roundings of sums of at most 5000 products, 2e-6 of the result at most;
    bf16: operands are rounded to 8 bits first, here and in the reference, so the same bound holds."""
    wl = NETS[name]
    net = lib.AlexNet(wl, batch, precision=precision, flags=lib.FLAG_DIRECT_CONV)
    rng = np.random.default_rng(batch)
    c, h = wl["in_c"], wl["crop"]
    for i, (co, k, st, pd, g, _, pool) in enumerate(wl["conv"], 1):
        ho = (h + 2 * pd - k) // st + 1
        x = rng.standard_normal((batch, c, h, h)).astype(np.float32)
        w = rng.standard_normal((co, c // g, k, k)).astype(np.float32)
        b = rng.standard_normal(co).astype(np.float32)
        dy = rng.standard_normal((batch, co, ho, ho)).astype(np.float32)
        if precision:  # exactly representable, so that rounding the operands changes nothing
            x, w, dy = (torch.from_numpy(a).bfloat16().float().numpy() for a in (x, w, dy))
        want = reference(x, w, b, dy, (k, st, pd, g))
        got = (net.conv_forward(i, cuda(x), cuda(w), cuda(b), False), net.conv_backward_data(i, cuda(dy), cuda(w), x.shape),
               net.conv_backward_weight(i, cuda(x), cuda(dy), w.shape)[0])
        for what, a, e in zip(("y", "dx", "dw"), got, want):
            a = a.cpu().numpy() if torch.is_tensor(a) else a
            assert rel_l2(a.reshape(e.shape), e) <= 2e-6, (i, what)
        c, h = co, (ho - 3) // 2 + 1 if pool else ho
    net.close()


def test_infinities_and_large_numbers(lib):
    """A tile whose split sums are not finite is computed again in fp32: infinities, NaNs and products past bf16's range come
    out where and as IEEE arithmetic has them, and the tiles beside them are untouched."""
    wl, batch = NETS["odd_channels"], 3
    net = lib.AlexNet(wl, batch, flags=lib.FLAG_DIRECT_CONV)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((batch, 20, 7, 7)).astype(np.float32)
    w = rng.standard_normal((36, 20, 3, 3)).astype(np.float32)
    b = np.zeros(36, np.float32)
    x[0, 3, 2, 2], x[1, 0, 4, 4], x[2, 7, 6, 0], x[2, 5, 3, 5] = np.inf, np.nan, 3e38, 1e-40
    with np.errstate(all="ignore"):
        want = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), padding=1).float().numpy()
    got = net.conv_forward(3, cuda(x), cuda(w), cuda(b), False)
    got = (got.cpu().numpy() if torch.is_tensor(got) else got).reshape(want.shape)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    ok = np.isfinite(want)
    assert np.abs(got[ok] - want[ok]).max() <= 1e-5 * np.abs(want[ok]).max()
    small = ok & (np.abs(want) < 1e3)
    assert rel_l2(got[small], want[small]) <= 2e-6
    net.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cin,cout,k,stride,crop", [(3, 6, 5, 2, 33), (3, 12, 7, 2, 37), (1, 4, 3, 1, 20), (2, 10, 3, 1, 14),
                                                    (3, 7, 2, 1, 9), (3, 9, 13, 2, 27)])
def test_pixels_beside_a_window_do_not_reach_it(lib, cin, cout, k, stride, crop, precision):
    """First layers in run mode, whose last quad of a kernel row reaches past the window: into the next pixels, the next row, the
    next picture.  Infinities and NaNs in every third picture come out where 64 bits have them and nowhere else."""
    rest = [(8, 3, 4, 1, 1, 0, 0), (8, 3, 4, 1, 1, 0, 0), (8, 3, 4, 1, 1, 0, 0), (8, 3, 1, 1, 1, 0, 0)]
    net, batch = lib.AlexNet(net_of([(cout, k, stride, 0, 1, 0, 0)] + rest, crop, [8, 8, 4], cin), 7, precision=precision), 7
    rng = np.random.default_rng(crop)
    x = rng.standard_normal((batch, cin, crop, crop)).astype(np.float32)
    w = rng.standard_normal((cout, cin, k, k)).astype(np.float32)
    if precision:
        x, w = (torch.from_numpy(a).bfloat16().float().numpy() for a in (x, w))
    for n in range(0, batch, 3):
        for at in ((0, 0), (0, crop - 1), (crop - 1, 0), tuple(rng.integers(0, crop, 2))):
            x[n, rng.integers(0, cin), at[0], at[1]] = rng.choice([np.inf, -np.inf, np.nan])
    with np.errstate(all="ignore"):
        want = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), stride=stride).numpy()
    got = net.conv_forward(1, cuda(x), cuda(w), None, False).cpu().numpy().reshape(want.shape)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    ok = np.isfinite(want)
    assert rel_l2(got[ok], want[ok]) <= 2e-6
    net.close()


@pytest.mark.parametrize("name,batch", [("odd_channels", 19), ("large_kernel", 9), ("one_pixel", 33), ("one_channel", 12),
                                        ("odd_channels", 150)])
def test_steps_on_edge_nets(lib, name, batch):
    """Two training steps against the oracle: paired gradients, slices put off to the end of the pass, no side stream."""
    run_step_and_compare(lib, NETS[name], batch, seed=31, bias=0.05, std=0.1, use_raw=False, steps=2, mom_std=0.01,
                          direct=False)


@pytest.mark.parametrize("wl,batch,precision", [(S.MINI, 16, 0), (S.MINI, 70, 1), (S.MIDI, 33, 0)])
def test_train_step_equals_its_parts(lib, wl, batch, precision):
    size, classes = wl["crop"], wl["fc"][-1]
    nets = [lib.AlexNet(wl, batch, seed=3, precision=precision) for _ in range(2)]
    rng = np.random.default_rng(9)
    p = {k: (rng.standard_normal(s) * 0.1).astype(np.float32) for k, s in nets[0].shapes.items()}
    for net in nets:
        net.set_params(p)
        net.set_momentum({k: v * 0.01 for k, v in p.items()})
    for step in range(3):
        x, labels = S.make_float_batch(batch, 3, size, size, classes, 20 + step)
        for net in nets:
            net.set_input(cuda(x), 0)
        la = float(nets[0].train_step(cuda(labels), step).cpu().item())
        lb = float(nets[1].forward_backward(cuda(labels), step).cpu().item())
        nets[1].apply_update()
        assert la == lb
    a, b = nets[0].get_params(), nets[1].get_params()
    assert all(np.array_equal(a[k], b[k]) for k in a)
    for net in nets:
        net.close()
