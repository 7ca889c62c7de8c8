"""Transformed 3x3 and 5x5 layers whose last tiles hold one output row and column (maps of 4n + 1, csrc/winograd.hip): row tiles
that end inside a range, one and several groups, tap products cut into slices, and maps of other sizes beside them."""
import numpy as np
import pytest
import torch

from helpers import rel_l2
from test_gpu_direct import net_of

pytestmark = pytest.mark.gpu

# Errors of the products of a transformed tile grow on the way to a value of the result, in mean square by
# sum_p A[p]^2 |G[p]|^2 |B[p]|^2 over the taps in each direction: a factor of 3.28, the same for all three passes.
GAIN = 3.28 ** 2


def bar(k):
    """An accumulator is rounded six times per 16 products (gemm_split.h), each time by 2^-24 of a partial sum that grows like
    the square root of its length; two for the transforms and the slices."""
    return GAIN * 2.0 ** -24 * (2.0 + np.sqrt(6.0 * k / 16.0))


@pytest.mark.parametrize("side,cin,cout,k,pad,groups,batch", [
    (13, 256, 384, 3, 1, 1, 37), (13, 384, 256, 3, 1, 2, 50), (9, 64, 200, 3, 1, 1, 70), (5, 256, 256, 3, 1, 1, 130),
    (17, 64, 96, 3, 1, 1, 20), (9, 128, 64, 5, 2, 2, 60), (11, 96, 132, 3, 2, 1, 40), (15, 100, 64, 3, 0, 1, 33),
    (14, 64, 64, 3, 1, 1, 40), (5, 8, 8, 3, 1, 1, 3)])
def test_all_passes_against_fp64(lib, side, cin, cout, k, pad, groups, batch):
    net = lib.AlexNet(net_of(side, cin, cout, k, pad, groups), batch)
    rng = np.random.default_rng(side)
    out = side + 2 * pad - k + 1
    x, w, dy, b = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)) for s in
                   ((batch, cin, side, side), (cout, cin // groups, k, k), (batch, cout, out, out), (cout,)))

    def close(got, want, terms):
        got = got.cpu().numpy().reshape(want.shape)
        assert rel_l2(got, want) <= bar(terms)
        assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong value
    n = ((k + 2) // 3) ** 2
    want = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=pad, groups=groups).relu().numpy()
    close(net.conv_forward(2, x.cuda(), w.cuda(), b.cuda(), True), want, n * cin // groups)
    want = torch.nn.functional.conv_transpose2d(dy.double(), w.double(), padding=pad, groups=groups).numpy()
    close(net.conv_backward_data(2, dy.cuda(), w.cuda(), x.shape), want, n * cout // groups)
    want = torch.nn.grad.conv2d_weight(x.double(), w.shape, dy.double(), padding=pad, groups=groups).numpy()
    close(net.conv_backward_weight(2, x.cuda(), dy.cuda(), w.shape)[0], want, batch * ((out + 3) // 4) ** 2)
    net.close()
