"""bf16 weight gradients read transposed from LDS (csrc/weight_direct.hip), through the operator of bf16 handles: row tiles
that end inside a tap and past the last one, column tiles that end inside a group, pixels that are no multiple of a k-tile and
end inside the first, the most taps a mask holds, strips of taps outside the picture on every side, and reductions in one and
in many slices."""
import numpy as np
import pytest
import torch

from helpers import rel_l2

pytestmark = pytest.mark.gpu


def net_of(side, cin, cout, k, pad, groups):
    """The layer under test as the second one, behind a pointwise first layer that makes its channels."""
    conv = [(cin, 1, 1, 0, 1, 0, 0), (cout, k, 1, pad, groups, 0, 0), (8, 3, 4, 1, 1, 0, 0), (8, 3, 4, 1, 1, 0, 0),
            (8, 3, 4, 1, 1, 0, 0)]
    return {"name": "weight_direct", "in_c": 8, "crop": side, "raw": side, "conv": conv, "fc": [8, 8, 4],
            "lrn": (5, 2.0, 1e-4, 0.75), "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9, "weight_decay": 5e-4}


@pytest.mark.parametrize("side,cin,cout,k,pad,groups,batch", [
    (13, 256, 384, 3, 1, 1, 40), (13, 384, 256, 3, 1, 2, 131), (27, 96, 256, 5, 2, 2, 37), (13, 384, 384, 3, 1, 2, 7),
    (9, 64, 200, 3, 2, 1, 71), (31, 72, 64, 1, 0, 1, 21), (14, 128, 72, 2, 1, 1, 50), (12, 56, 120, 5, 4, 1, 90),
    (11, 192, 192, 3, 1, 1, 3), (8, 512, 512, 3, 1, 4, 130), (7, 1024, 1024, 1, 0, 1, 1), (10, 40, 40, 3, 1, 1, 200)])
def test_weight_gradient_against_fp64(lib, side, cin, cout, k, pad, groups, batch):
    """Operands are bf16 numbers already, so that only fp32 sums are rounded: of up to 27000 products here, in slices of at
    most 7000, each term's rounding independent, sqrt(7000) * 2^-24 = 5e-6 of the result."""
    net = lib.AlexNet(net_of(side, cin, cout, k, pad, groups), batch, precision=1)
    rng = np.random.default_rng(side)
    out = side + 2 * pad - k + 1
    x, dy = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float() for s in
             ((batch, cin, side, side), (batch, cout, out, out)))
    shape = (cout, cin // groups, k, k)
    want = torch.nn.grad.conv2d_weight(x.double(), shape, dy.double(), padding=pad, groups=groups).numpy()
    got = net.conv_backward_weight(2, x.cuda(), dy.cuda(), shape)
    got = (got[0] if isinstance(got, (tuple, list)) else got).cpu().numpy().reshape(shape)
    assert rel_l2(got, want) <= 5e-6
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong tap
    net.close()
