"""The first layer's bf16 product with weights and picture rows in LDS (csrc/first_layer.hip): strides 2, 4 and 6 (one to
three planes), one to four blocks of channels, kernels whose octets are even and odd in number, rows of odd width, tiles that
end inside a picture, one, two and three picture channels -- and geometries that do not fit and run as a gather GEMM."""
import numpy as np
import pytest
import torch

from gpu_common import cuda
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def net_of(in_c, crop, cout, k, stride):
    rest = [(16, 3, 4, 1, 1, 0, 0), (16, 3, 4, 1, 1, 0, 0), (16, 3, 4, 1, 1, 0, 0), (8, 3, 1, 1, 1, 0, 0)]
    return {"name": "first", "in_c": in_c, "crop": crop, "raw": crop, "conv": [(cout, k, stride, 0, 1, 0, 1)] + rest,
            "fc": [16, 8, 4], "lrn": (5, 2.0, 1e-4, 0.75), "dropout_p": 0.5, "lr": 0.01, "momentum": 0.9,
            "weight_decay": 5e-4}


@pytest.mark.parametrize("in_c,crop,cout,k,stride,batch", [
    (3, 227, 96, 11, 4, 5), (3, 131, 128, 7, 2, 24), (1, 200, 40, 5, 4, 60), (2, 253, 8, 15, 6, 40), (3, 515, 64, 3, 2, 5),
    (3, 160, 72, 9, 2, 12), (3, 227, 136, 11, 4, 5), (3, 300, 32, 3, 1, 2), (3, 199, 48, 6, 3, 9)])
def test_first_layer_against_fp64(lib, in_c, crop, cout, k, stride, batch):
    """Operands are bf16 numbers already, so that only fp32 sums of at most 675 products are rounded: 2e-6 of the result."""
    net = lib.AlexNet(net_of(in_c, crop, cout, k, stride), batch, precision=1)
    rng = np.random.default_rng(k)
    x, w = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).bfloat16().float()
            for s in ((batch, in_c, crop, crop), (cout, in_c, k, k)))
    b = torch.from_numpy(rng.standard_normal(cout).astype(np.float32))
    for relu in (False, True):
        want = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), stride=stride)
        want = (want.relu() if relu else want).numpy()
        got = net.conv_forward(1, x.cuda(), w.cuda(), b.cuda(), relu).cpu().numpy().reshape(want.shape)
        assert rel_l2(got, want) <= 2e-6
        assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()  # no single wrong pixel
    net.close()


@pytest.mark.parametrize("in_c,crop,cout,k,stride,batch", [
    (3, 131, 96, 11, 4, 24), (3, 160, 72, 9, 2, 12), (1, 200, 40, 5, 4, 60), (2, 253, 8, 15, 6, 40), (3, 227, 136, 11, 4, 5)])
def test_infinities_reach_their_own_windows_only(lib, in_c, crop, cout, k, stride, batch):
    """The rows of a tile past a picture's end come from the next picture and must not show.  A kernel row is read in pairs of
    pixels: behind an odd one the next pixel in memory, at a row's end the next row's first, meets zero weights, so that an
    infinity there makes a NaN.  That much and no more: the reference has the same extra column, everything else is as it is
    without infinities, bit for bit."""
    net = lib.AlexNet(net_of(in_c, crop, cout, k, stride), batch, precision=1)
    rng = np.random.default_rng(2)
    x = rng.standard_normal((batch, in_c, crop, crop)).astype(np.float32)
    w = cuda(rng.standard_normal((cout, in_c, k, k)).astype(np.float32))
    clean = net.conv_forward(1, cuda(x), w, None).cpu().numpy()
    x[batch // 3] = np.inf
    for n in (0, batch - 1):
        for at in ((0, 0), (0, crop - 1), (crop - 1, 0), tuple(rng.integers(0, crop, 2))):
            x[n, rng.integers(0, in_c), at[0], at[1]] = rng.choice([np.inf, -np.inf, np.nan])
    got = net.conv_forward(1, cuda(x), w, None).cpu().numpy()
    xt, wt = torch.from_numpy(x).bfloat16().double(), w.cpu().bfloat16().double()
    if k % 2:
        rows = xt.permute(1, 0, 2, 3).reshape(in_c, -1, crop)
        behind = torch.cat([rows[:, 1:, :1], torch.zeros(in_c, 1, 1, dtype=torch.double)], 1)
        xt = torch.cat([rows, behind], 2).reshape(in_c, batch, crop, crop + 1).permute(1, 0, 2, 3)
        wt = torch.nn.functional.pad(wt, (0, 1))
    # the reference multiplies its zero weights too: one product after the other, as F.conv2d need not
    cols = torch.nn.functional.unfold(xt, (k, k + k % 2), stride=stride)
    want = torch.matmul(wt.flatten(1), cols).numpy().reshape(got.shape)
    finite = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)].astype(np.float32))
    got, clean = (a.reshape(batch, -1) for a in (got, clean))
    finite = finite.reshape(batch, -1)
    assert finite.any() and not finite.all()
    assert np.array_equal(got[finite], clean[finite])
    net.close()
