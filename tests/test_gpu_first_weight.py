"""The first layer's bf16 weight gradient with the whole gradient in a workgroup's accumulators (csrc/first_weight.hip): one to
three picture channels, strides 1 to 4, kernels that are no multiple of four taps, rows of 12 to 64 outputs, column blocks that
are partly empty, runs of rows that start and end inside a picture, one picture, and infinities at a picture's edge."""
import numpy as np
import pytest
import torch

from helpers import rel_l2

pytestmark = pytest.mark.gpu


def net_of(in_c, crop, cout, k, stride):
    rest = [(16, 3, 4, 1, 1, 0, 0), (16, 3, 4, 1, 1, 0, 0), (16, 3, 4, 1, 1, 0, 0), (8, 3, 1, 1, 1, 0, 0)]
    return {"name": "first_weight", "in_c": in_c, "crop": crop, "raw": crop, "conv": [(cout, k, stride, 0, 1, 0, 1)] + rest,
            "fc": [16, 8, 4], "lrn": (5, 2.0, 1e-4, 0.75), "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9,
            "weight_decay": 5e-4}


def inputs(in_c, crop, cout, k, stride, batch):
    rng = np.random.default_rng(k)
    out = (crop - k) // stride + 1
    return [torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float()
            for s in ((batch, in_c, crop, crop), (batch, cout, out, out))]


@pytest.mark.parametrize("in_c,crop,cout,k,stride,batch", [
    (3, 227, 96, 11, 4, 5), (3, 227, 96, 11, 4, 1), (3, 131, 96, 7, 2, 24), (1, 200, 40, 5, 4, 60), (2, 66, 8, 3, 1, 30),
    (3, 250, 72, 12, 4, 9), (3, 41, 48, 6, 3, 70)])
def test_first_layer_weight_gradient_against_fp64(lib, in_c, crop, cout, k, stride, batch):
    """Operands are bf16 numbers already, so that only fp32 sums are rounded: slices of at most 12 output rows, 588 products, and
    256 slices; (sqrt(588) + sqrt(256)) * 2^-24 = 2.4e-6 of the result."""
    net = lib.AlexNet(net_of(in_c, crop, cout, k, stride), batch, precision=1)
    x, dy = inputs(in_c, crop, cout, k, stride, batch)
    shape = (cout, in_c, k, k)
    cols = torch.nn.functional.unfold(x.double(), k, stride=stride)  # [batch][(c, r, s)][pixel]
    want = torch.matmul(dy.double().flatten(2), cols.transpose(1, 2).contiguous()).sum(0).view(shape).numpy()
    got = net.conv_backward_weight(1, x.cuda(), dy.cuda(), shape)[0].cpu().numpy()
    assert rel_l2(got, want) <= 2.4e-6
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong tap
    net.close()


def test_an_infinity_reaches_its_own_taps_only(lib):
    """The last column of a picture is under the last output pixel's last tap and no other: outputs past the row's end, which
    fill the last step of the reduction, must not multiply it."""
    geo = (3, 227, 96, 11, 4, 3)
    net = lib.AlexNet(net_of(*geo[:5]), geo[5], precision=1)
    x, dy = inputs(*geo)
    clean = net.conv_backward_weight(1, x.cuda(), dy.cuda(), (96, 3, 11, 11))[0].cpu().numpy()
    x[1, 2, 100, 226] = float("inf")
    got = net.conv_backward_weight(1, x.cuda(), dy.cuda(), (96, 3, 11, 11))[0].cpu().numpy()
    hit = np.zeros((96, 3, 11, 11), bool)
    hit[:, 2, 0::4, 10] = True
    assert not np.isfinite(got[hit]).any()
    assert np.array_equal(got[~hit], clean[~hit])
    net.close()
