"""Forward products from pictures in LDS (csrc/patch_conv.hip): both tiles, bands of unequal height, pictures of one band, paddings
that put whole taps outside, even kernels, 16 and 48 channels per group, several column tiles, a single tap."""
import numpy as np
import pytest
import torch

from helpers import rel_l2
from test_gpu_direct import net_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,cin,cout,k,pad,groups,batch", [
    (27, 96, 256, 5, 2, 2, 32), (27, 96, 256, 5, 2, 2, 128), (13, 48, 128, 3, 1, 1, 300), (13, 48, 256, 3, 0, 1, 257),
    (30, 32, 256, 3, 1, 2, 40), (30, 16, 128, 4, 3, 1, 300), (20, 96, 768, 6, 1, 2, 40), (60, 48, 128, 2, 1, 1, 30),
    (14, 16, 128, 1, 0, 1, 260), (11, 48, 128, 7, 6, 1, 140),
    (27, 96, 256, 5, 2, 2, 64), (13, 48, 128, 3, 1, 1, 512), (50, 48, 256, 3, 1, 1, 17)])
def test_forward_against_fp64(lib, side, cin, cout, k, pad, groups, batch):
    """Operands are bf16 numbers already: only fp32 sums of at most 2352 products are rounded, 3e-6 of the result."""
    net = lib.AlexNet(net_of(side, cin, cout, k, pad, groups), batch, precision=1)
    rng = np.random.default_rng(side)
    x, w = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float() for s in
            ((batch, cin, side, side), (cout, cin // groups, k, k)))
    b = torch.from_numpy(rng.standard_normal(cout).astype(np.float32))
    for relu in (True, False):
        want = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=pad, groups=groups)
        want = (want.relu() if relu else want).numpy()
        got = net.conv_forward(2, x.cuda(), w.cuda(), b.cuda(), relu).cpu().numpy().reshape(want.shape)
        assert rel_l2(got, want) <= 3e-6
        assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong pixel
    net.close()
