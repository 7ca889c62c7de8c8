"""Stored and floating-point pictures on their way to channel-last rows, and the first layer that reads them, at channel
counts, widths and kernel sizes beside those of the nets."""
import numpy as np
import pytest

import synthetic_inputs as S
from gpu_common import build_pair, cuda
from helpers import rel_l2
from oracle import alexnet_oracle as O
from test_gpu_bf16 import EXACT_RTOL, round_bf16

pytestmark = pytest.mark.gpu


def net_of(channels, crop, raw, k, stride):
    return dict(S.MINI, name="pictures", in_c=channels, crop=crop, raw=raw,
                conv=[(16, k, stride, 0, 1, 0, 0), (16, 3, 2, 1, 1, 0, 0), (16, 3, 2, 1, 1, 0, 0)] + [(16, 3, 1, 1, 1, 0, 0)] * 2,
                fc=[16, 8, 5])


@pytest.mark.parametrize("shape", [(2, 1, 33, 35), (3, 3, 32, 32), (2, 3, 31, 37), (1, 1, 1, 1), (2, 3, 1, 3), (1, 3, 64, 65)])
def test_pictures_to_channel_last_rows(lib, shape):
    """One and three channels, pixel counts below, at and past a workgroup's 1024 and no multiple of four."""
    x = S.make_normal(shape, 1)
    assert np.array_equal(lib.nchw_to_nhwc(cuda(x)).cpu().numpy(), np.transpose(x, (0, 2, 3, 1)))


# widths below the wide kernel's line (128), at it, no multiple of four, one and two passes of 256 pixels through LDS
@pytest.mark.parametrize("channels", [1, 2, 3])
@pytest.mark.parametrize("crop,raw", [(127, 130), (128, 128), (131, 140), (256, 259), (301, 306), (515, 515)])
@pytest.mark.parametrize("precision", [0, 1])
def test_preprocess_crop_mirror_exact(lib, channels, crop, raw, precision):
    batch = 3
    wl = net_of(channels, crop, raw, 7, 4)
    net, spec, p64, _ = build_pair(lib, wl, batch, seed=5, bias=0.1, std=0.05, precision=precision)
    pictures, labels = S.make_raw_batch(batch, channels, raw, raw, 5, 7)
    mean = S.make_mean_image(channels, raw, raw, 8)
    flips = set()
    for step in (0, 1, 2, 3):
        net.preprocess(cuda(pictures), cuda(mean), step, step % 2)
        ox, oy, flip = O.crop_flip_params(spec, step)
        flips |= set(flip.tolist())
        want = O.preprocess(pictures, mean, ox, oy, flip, crop, crop).astype(np.float32)
        assert np.array_equal(net.tensor(lib.T_INPUT, step % 2).reshape(want.shape), want)
    assert flips == {0, 1}
    # what the first layer makes of it: bf16 handles read the padded copy that came out of the same pass
    net.forward_backward(cuda(labels), step, slot=step % 2)
    act = net.tensor(lib.T_CONV_ACT, 1)
    rounded = round_bf16 if precision else lambda a: np.asarray(a, np.float64)
    ref = np.maximum(O.conv_forward(rounded(want), rounded(p64["conv1.w"]), p64["conv1.b"], 4, 0, 1), 0)
    assert rel_l2(act.reshape(ref.shape), ref) <= EXACT_RTOL
    net.close()


# kernel rows of 24, 18, 21 and 16 floats: none, two, one and none left over behind the whole quads; nine floats, a run too
# short for the split kernels; rows of 16 pixels and one more than 16
@pytest.mark.parametrize("channels,k,crop,stride", [(3, 8, 46, 2), (3, 6, 37, 2), (3, 7, 38, 1), (1, 16, 47, 2), (3, 3, 40, 2),
                                                    (3, 6, 36, 2), (1, 18, 50, 2)])
def test_first_layer_with_other_kernels(lib, channels, k, crop, stride):
    batch = 3
    wl = net_of(channels, crop, crop, k, stride)
    net = lib.AlexNet(wl, batch)
    out = (crop - k) // stride + 1
    x, dy = S.make_normal((batch, channels, crop, crop), 21), S.make_normal((batch, 16, out, out), 22)
    w, b = S.make_normal((16, channels, k, k), 23, std=0.1), S.make_normal((16,), 24)
    y = net.conv_forward(1, x, w, b).cpu().numpy().reshape(dy.shape)
    assert rel_l2(y, O.conv_forward(x, w, b, stride, 0, 1)) <= EXACT_RTOL
    dw, db = net.conv_backward_weight(1, x, dy, w.shape)
    want_w, want_b = O.conv_backward_weight(x, dy, k, stride, 0, 1)
    assert rel_l2(dw.cpu().numpy(), want_w) <= EXACT_RTOL and rel_l2(db.cpu().numpy(), want_b) <= EXACT_RTOL
    net.close()
