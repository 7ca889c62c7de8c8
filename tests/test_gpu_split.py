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


def test_bf16_products_with_192_columns(lib):
    """The 128 x 192 bf16 tile (csrc/gemm16.h): 545 row tiles, the last one ragged, padding on every side, forward and
    data gradient, against the fp32 products of the same bf16 values (fp32 sums on both sides)."""
    wl = dict(S.MINI, name="wide", crop=33, raw=33,
              conv=[(192, 1, 1, 0, 1, 0, 0), (192, 3, 1, 1, 1, 0, 0)] + [(8, 1, 1, 0, 1, 0, 0)] * 3, fc=[8, 8, 4])
    batch = 64
    bf, ref = lib.AlexNet(wl, batch, precision=1), lib.AlexNet(wl, batch, flags=lib.FLAG_DIRECT_CONV)

    def values(shape, seed):  # bf16 holds these exactly
        v = S.make_normal(shape, seed)
        return (v.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    x, w = values((batch, 192, 33, 33), 1), values((192, 192, 3, 3), 2)
    dy, b = values((batch, 192, 33, 33), 3), np.zeros(192, np.float32)
    for op in (lambda n: n.conv_forward(2, x, w, b), lambda n: n.conv_backward_data(2, dy, w, x.shape)):
        assert rel_l2(op(bf).cpu().numpy(), op(ref).cpu().numpy()) <= _bar(9 * 192)
    bf.close()
    ref.close()


@pytest.mark.parametrize("batch,nin,nout", [(1, 8, 8), (3, 1032, 24), (4, 2048, 9)])
def test_few_dense_rows_with_bf16_products(lib, batch, nin, nout):
    """Dense layers on a few rows of a bf16 handle: both operands rounded to bf16, fp32 sums."""
    net = lib.AlexNet(dict(S.MINI, name="rows", fc=[nin, nout, 4]), batch, precision=1)

    def values(shape, seed):  # bf16 holds these exactly
        return (S.make_normal(shape, seed).view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    x, w, b = values((batch, nin), 1), values((nout, nin), 2), S.make_normal((nout,), 3)
    y = net.fc_forward(7, x, w, b).cpu().numpy()
    assert rel_l2(y, x.astype(np.float64) @ w.astype(np.float64).T + b) <= _bar(nin)
    net.close()


def _fp32_matrix_order(a, b):
    """a^T b with the sum rounded to fp32 after every two products, as the fp32 matrix instructions do."""
    s = np.zeros((a.shape[1], b.shape[1]), np.float32)
    for k in range(0, len(a), 2):
        s = (s + a[k:k + 2].astype(np.float64).T @ b[k:k + 2].astype(np.float64)).astype(np.float32)
    return s


@pytest.mark.parametrize("kind", ["normal", "relu", "positive"])
@pytest.mark.parametrize("batch", [16, 20, 32, 64, 200])
def test_no_further_from_the_exact_sum_than_fp32_products(lib, batch, kind):
    """The weight gradient of a dense layer (one reduction over the batch, no slices) against float64, and as far as
    that from it the same product summed as the fp32 matrix instructions sum it.  Behind a ReLU half the products are
    zero and their additions exact, where a term product of the split is rounded all the same."""
    n = 128
    net = lib.AlexNet(dict(S.MINI, name="sums", fc=[n, n, 4]), batch)
    x, dy = S.make_normal((batch, n), 11), S.make_normal((batch, n), 12)
    if kind == "relu":
        x = np.maximum(x, 0)
    if kind == "positive":
        x, dy = 1 + np.abs(x) % 1, 1 + np.abs(dy) % 1
    _, dw, _ = net.fc_backward(7, x, np.zeros((n, n), np.float32), dy)
    exact = dy.astype(np.float64).T @ x.astype(np.float64)
    assert rel_l2(dw.cpu().numpy(), exact) <= rel_l2(_fp32_matrix_order(dy, x), exact)
    net.close()


def test_products_of_single_values_are_correctly_rounded(lib):
    """A reduction over one value is one multiplication: the result is the product rounded once, bit for bit -- the
    weight gradients of a dense layer and of a 1x1 layer on 1x1 maps at a batch of one."""
    wl = dict(S.MINI, name="ones", crop=1, raw=1, conv=[(8, 1, 1, 0, 1, 0, 0)] * 5, fc=[64, 132, 4])
    net = lib.AlexNet(wl, 1)
    x, dy = S.make_normal((1, 64), 21), S.make_normal((1, 132), 22)
    _, dw, _ = net.fc_backward(7, x, np.zeros((132, 64), np.float32), dy)
    assert np.array_equal(dw.cpu().numpy(), dy.T * x)
    x, dy = S.make_normal((1, 8, 1, 1), 23), S.make_normal((1, 8, 1, 1), 24)
    dw, _ = net.conv_backward_weight(2, x, dy, (8, 8, 1, 1))
    assert np.array_equal(dw.cpu().numpy().reshape(8, 8), dy.reshape(8, 1) * x.reshape(1, 8))
    net.close()


def _same_values(got, exact, k):
    """Infinities and NaNs where and as fp32 sums have them, everything else within the bar."""
    with np.errstate(over="ignore"):
        want = exact.astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    scale = np.abs(exact[fin]).max()  # magnitudes up to the largest fp32 number
    assert rel_l2(got[fin] / scale, exact[fin] / scale) <= _bar(k)


# value of one operand element, of the others it is multiplied with: an infinity, a NaN, a finite value that rounds to
# infinity as bf16, a product of two such roundings beyond the fp32 range where the product itself is not
@pytest.mark.parametrize("value,other", [(np.inf, 1.0), (-np.inf, 1.0), (np.nan, 1.0), (3.4e38, 1e-3),
                                         (1.9999 * 2.0 ** 63, 2.0 ** 63.5)])
@pytest.mark.parametrize("batch,n", [(8, 64), (130, 100)])
def test_operands_that_are_not_finite_or_close_to_overflow(lib, batch, n, value, other):
    net = lib.AlexNet(dict(S.MINI, name="range", fc=[n, n, 4]), batch)
    x, w = np.abs(S.make_normal((batch, n), 31)) + 0.5, np.abs(S.make_normal((n, n), 32)) + 0.5
    x[3, 5] = value
    w[:, 5] = np.where(np.arange(n) % 7 == 0, 0, w[:, 5] * other)  # inf * 0 is NaN
    zero = np.zeros(n, np.float32)
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    with np.errstate(invalid="ignore"):
        y, dx, dw = x64 @ w64.T, x64 @ w64, x64.T @ x64
    _same_values(net.fc_forward(7, x, w, zero).cpu().numpy(), y, n)
    with np.errstate(invalid="ignore"):
        _same_values(net.fc_forward(7, x, w, zero, relu=True).cpu().numpy(), np.where(y > 0, y, 0), n)
    gx, gw, _ = net.fc_backward(7, x, w, x)  # the gradient of the layer is x too
    _same_values(gx.cpu().numpy(), dx, n)
    _same_values(gw.cpu().numpy(), dw, batch)
    net.close()


def test_first_layer_with_infinite_pictures(lib):
    """The first layer's products (runs of whole kernel rows): an infinite pixel reaches the outputs whose window holds
    it as an infinity, and no other."""
    wl = dict(S.MINI, name="pictures", crop=41, raw=41)
    net = lib.AlexNet(wl, 2)
    x, w = np.abs(S.make_normal((2, 3, 41, 41), 41)) + 0.5, np.abs(S.make_normal((16, 3, 7, 7), 42)) + 0.5
    x[1, 2, 20, 20] = np.inf
    y = net.conv_forward(1, x, w, None, relu=True).cpu().numpy().reshape(2, 16, 18, 18)
    hit = np.zeros(y.shape, bool)
    hit[1, :, 7:11, 7:11] = True  # windows 2q .. 2q + 6 that hold 20
    assert np.array_equal(np.isinf(y), hit) and not np.isnan(y).any()
    dy = np.abs(S.make_normal((2, 16, 18, 18), 43)) + 0.5
    dw, _ = net.conv_backward_weight(1, x, dy, w.shape)
    dw = dw.cpu().numpy()
    hit = np.zeros(dw.shape, bool)
    hit[:, 2, 0::2, 0::2] = True  # 20 = 2q + r for an even r
    assert np.array_equal(np.isinf(dw), hit) and not np.isnan(dw).any()
    net.close()


@pytest.mark.parametrize("size", [1e-33, 1e-36, 1e-38])
def test_operands_close_to_the_smallest_normal_numbers(lib, size):
    """Values down to 2^-126: every one of their 24 bits counts."""
    batch, n = 40, 64
    net = lib.AlexNet(dict(S.MINI, name="small", fc=[n, n, 4]), batch)
    x, w, dy = (S.make_normal(s, 51 + i) for i, s in enumerate([(batch, n), (n, n), (batch, n)]))
    x = (np.sign(x) * (1 + np.abs(x)) * size * 1.2).astype(np.float32)
    w, dy = 64 * w, 64 * dy  # the sums themselves stay normal numbers
    x64, w64, dy64 = (a.astype(np.float64) for a in (x, w, dy))
    y = net.fc_forward(7, x, w, np.zeros(n, np.float32)).cpu().numpy()
    assert rel_l2(y / size, x64 @ w64.T / size) <= _bar(n)
    _, dw, _ = net.fc_backward(7, x, w, dy)
    assert rel_l2(dw.cpu().numpy() / size, dy64.T @ x64 / size) <= _bar(batch)
    net.close()


@pytest.mark.parametrize("batch,nin,nout", [(1, 8, 8), (2, 260, 12), (4, 2048, 9)])
def test_few_dense_rows_round_both_operands_to_bf16(lib, batch, nin, nout):
    """Operands with all their bits: the result is the fp32 sum of the operands rounded to the nearest bf16, ties to even,
    and neither the unrounded product nor that of values cut off."""
    def nearest(a):
        u = a.view(np.uint32).astype(np.uint64)
        return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32).astype(np.float64)

    def cut(a):
        return (a.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32).astype(np.float64)
    net = lib.AlexNet(dict(S.MINI, name="rows", fc=[nin, nout, 4]), batch, precision=1)
    x, w, b = S.make_normal((batch, nin), 61), S.make_normal((nout, nin), 62), np.zeros(nout, np.float32)
    x[:, 0] = np.float32(1 + 2.0 ** -8)  # ties: down to 1, up to 1 + 2^-6
    w[:, 1] = np.float32(1 + 3 * 2.0 ** -8)
    y = net.fc_forward(7, x, w, b).cpu().numpy()
    assert rel_l2(y, nearest(x) @ nearest(w).T) <= _bar(nin)
    assert rel_l2(y, cut(x) @ cut(w).T) > 1e-4 and rel_l2(y, x.astype(np.float64) @ w.astype(np.float64).T) > 1e-4
    net.close()
