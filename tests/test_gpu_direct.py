"""bf16 products with operands loaded to LDS directly (csrc/gemm_direct.h), through the convolution operators of bf16 handles:
row and column tiles that end inside a picture and inside a group, taps that fall outside on every side, one and many taps,
channels that are multiples of 64 (a k-tile inside one tap) and of eight (an octet inside one), an odd number of k-tiles and
a single one, reductions in slices, and more taps than a lane's mask has bits (which stay with the other kernels)."""
import numpy as np
import pytest
import torch

from helpers import rel_l2

pytestmark = pytest.mark.gpu


def net_of(side, cin, cout, k, pad, groups):
    """A layer under test as the second one, behind a pointwise first layer that makes its channels."""
    conv = [(cin, 1, 1, 0, 1, 0, 0), (cout, k, 1, pad, groups, 0, 0), (8, 3, 4, 1, 1, 0, 0), (8, 3, 4, 1, 1, 0, 0),
            (8, 3, 4, 1, 1, 0, 0)]
    return {"name": "direct", "in_c": 8, "crop": side, "raw": side, "conv": conv, "fc": [8, 8, 4], "lrn": (5, 2.0, 1e-4, 0.75),
            "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9, "weight_decay": 5e-4}


@pytest.mark.parametrize("side,cin,cout,k,pad,groups,batch", [
    (13, 256, 384, 3, 1, 1, 40), (13, 384, 256, 3, 1, 2, 130), (27, 96, 256, 5, 2, 2, 37), (9, 64, 200, 3, 2, 1, 70),
    (31, 64, 64, 1, 0, 1, 21), (14, 128, 72, 2, 1, 1, 50), (12, 56, 120, 4, 0, 1, 90), (11, 192, 192, 3, 1, 1, 3),
    (16, 64, 128, 6, 3, 1, 30), (8, 512, 512, 3, 1, 4, 130)])
def test_forward_and_data_gradient_against_fp64(lib, side, cin, cout, k, pad, groups, batch):
    """Operands are bf16 numbers already, so that only fp32 sums of at most 3456 products are rounded: 3e-6 of the result."""
    net = lib.AlexNet(net_of(side, cin, cout, k, pad, groups), batch, precision=1)
    rng = np.random.default_rng(side)
    out = side + 2 * pad - k + 1
    x, w, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float() for s in
                ((batch, cin, side, side), (cout, cin // groups, k, k), (batch, cout, out, out)))
    b = torch.from_numpy(rng.standard_normal(cout).astype(np.float32))
    want = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=pad, groups=groups).relu().numpy()
    got = net.conv_forward(2, x.cuda(), w.cuda(), b.cuda(), True).cpu().numpy().reshape(want.shape)
    assert rel_l2(got, want) <= 3e-6
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong pixel
    want = torch.nn.functional.conv_transpose2d(dy.double(), w.double(), padding=pad, groups=groups).numpy()
    got = net.conv_backward_data(2, dy.cuda(), w.cuda(), x.shape).cpu().numpy()
    assert rel_l2(got, want) <= 3e-6
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()
    net.close()
