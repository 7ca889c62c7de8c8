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


def test_pictures_next_to_each_other_do_not_mix(lib):
    """One picture full of infinities: the rows of a tile past a picture's end, and the padded pixels, come from others."""
    wl, batch = net_of(3, 131, 96, 11, 4), 24
    net = lib.AlexNet(wl, batch, precision=1)
    rng = np.random.default_rng(2)
    x = rng.standard_normal((batch, 3, 131, 131)).astype(np.float32)
    w = cuda(rng.standard_normal((96, 3, 11, 11)).astype(np.float32))
    clean = net.conv_forward(1, cuda(x), w, None).cpu().numpy().reshape(batch, -1)
    x[7] = np.inf
    got = net.conv_forward(1, cuda(x), w, None).cpu().numpy().reshape(batch, -1)
    keep = np.arange(batch) != 7
    assert np.isfinite(got[keep]).mean() > 0.99 and not np.isfinite(got[7]).any()
    same = np.isfinite(got[keep])
    assert np.array_equal(got[keep][same], clean[keep][same])
    net.close()
