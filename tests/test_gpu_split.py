"""fp32 products on the bf16 matrix cores (csrc/gemm_split.h) at the edges of their tiles and k-tiles, through the
dense layers' entry points, against float64."""
import numpy as np
import pytest

import synthetic_inputs as S
from gpu_common import cuda
from helpers import rel_l2

pytestmark = pytest.mark.gpu


def _bar(k):
    """An accumulator is rounded six times per 16 products, each time by at most 2^-24 of a partial sum that grows
    like the square root of its length: 2^-24 * sqrt(6k/16) on average signs, and as much again for the slices and
    the terms that are dropped."""
    return 2.0 ** -24 * (2.0 + 2.0 * np.sqrt(6.0 * k / 16.0))


# batch, in, out: one quad, tiles just filled, one quad past a tile of 64 / 96 / 128 / 192, k below and at a k-tile,
# reductions cut into slices, an odd batch (the reduction of the weight gradient)
@pytest.mark.parametrize("batch,nin,nout", [(1, 4, 4), (3, 16, 20), (37, 132, 196), (128, 128, 192), (129, 260, 100),
                                            (64, 4096, 64), (33, 2052, 1000)])
def test_dense_products_at_tile_edges(lib, batch, nin, nout):
    wl = dict(S.MINI, name="edges", fc=[nin, nout, 4])
    net = lib.AlexNet(wl, batch)
    x, w = S.make_normal((batch, nin), 1), S.make_normal((nout, nin), 2)
    b, dy = S.make_normal((nout,), 3), S.make_normal((batch, nout), 4)
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    y = net.fc_forward(7, x, w, b).cpu().numpy()
    assert rel_l2(y, x64 @ w64.T + b) <= _bar(nin)
    dx, dw, _ = net.fc_backward(7, x, w, dy)
    assert rel_l2(dx.cpu().numpy(), dy64 @ w64) <= _bar(nout)
    assert rel_l2(dw.cpu().numpy(), dy64.T @ x64) <= _bar(batch)
    net.close()


def test_wide_range_of_magnitudes(lib):
    """Operand values over 2^-60 .. 2^60 with all 24 significand bits in use: no term of the split is lost."""
    rng = np.random.default_rng(5)
    batch, n = 32, 128
    net = lib.AlexNet(dict(S.MINI, name="range", fc=[n, n, 4]), batch)
    sx, sw = 2.0 ** rng.integers(-60, 60, (batch, 1)), 2.0 ** rng.integers(-60, 60, (n, 1))
    x, w = (S.make_normal((batch, n), 6) * sx).astype(np.float32), (S.make_normal((n, n), 7) * sw).astype(np.float32)
    y = net.fc_forward(7, x, w, np.zeros(n, np.float32)).cpu().numpy()
    scale = sx * sw.T  # every output on its own scale
    assert rel_l2(y / scale, (x.astype(np.float64) @ w.T.astype(np.float64)) / scale) <= _bar(n)
    net.close()
