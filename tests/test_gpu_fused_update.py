"""Dense weight gradients that update their weights where they are summed up (EpiSgd): the same bits as the gradient and the
update one after the other, at ragged widths, on tiles just filled and batches of a k-tile and its neighbours."""
import numpy as np
import pytest

import synthetic_inputs as S
from gpu_common import build_pair, cuda

pytestmark = pytest.mark.gpu


def steps_are_equal(lib, widths, batch, precision):
    """Two steps of two replicas, one by train_step(), one by gradient and update; the profile of the last train_step()."""
    wl = dict(S.MIDI, name="update", fc=list(widths))
    a, b = (build_pair(lib, wl, batch, seed=S.SEED_BASE + 4, pseed=4, std=0.05, bias=0.1, mom_std=0.01, precision=precision)[0]
            for _ in range(2))
    mean = cuda(S.make_mean_image(3, wl["raw"], wl["raw"], S.SEED_BASE + 7))
    for step in range(2):
        raw, labels = (cuda(t) for t in S.make_raw_batch(batch, 3, wl["raw"], wl["raw"], widths[-1], S.SEED_BASE + 40 + step))
        a.preprocess(raw, mean, step, step % 2)
        b.preprocess(raw, mean, step, step % 2)
        lib.profile_begin()
        la = a.train_step(labels, step, slot=step % 2).cpu()
        seen = {e["name"]: e for e in lib.profile_end()}
        lb = b.forward_backward(labels, step, slot=step % 2).cpu()
        b.apply_update()
        assert la.item() == lb.item()
    for pa, pb in ((a.get_params(), b.get_params()), (a.get_momentum(), b.get_momentum())):
        for k in pa:
            assert np.isfinite(pa[k]).all() and np.array_equal(pa[k], pb[k]), k
    a.close()
    b.close()
    return seen


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("widths,batch", [((132, 68, 20), 33), ((128, 256, 64), 32), ((264, 72, 1000), 8), ((8, 8, 4), 65),
                                          ((201, 135, 37), 16)])
def test_train_step_equals_gradient_and_update(lib, precision, widths, batch):
    steps_are_equal(lib, widths, batch, precision)


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("widths,batch,layers", [
    ((2048, 2048, 1000), 64, (7, 8)), ((2056, 1992, 1016), 63, (7, 8)), ((2048, 1928, 1000), 65, (7, 8)),
    ((4096, 2056, 1000), 15, (7,)), ((4104, 2048, 1000), 16, (7,)), ((4096, 2184, 1000), 17, (7,)),
    ((4096, 4096, 1000), 129, (6, 7, 8)), ((2048, 3080, 1000), 200, (7, 8))])
def test_products_that_update(lib, precision, widths, batch, layers):
    """Layers too large for a small product: the profile shows that their gradients' launches read and wrote weights and momentum
    too (five tensors of the weights' size), 2056 or 1992 columns end inside a tile and inside a wave's blocks."""
    seen = steps_are_equal(lib, widths, batch, precision)
    dims = [40, *widths]  # the small convolutions leave 40 values
    for layer in layers:
        fin, fout = dims[layer - 6:layer - 4]
        e = seen["fc%d.bwd_w:%s" % (layer, "gemm_bf16" if precision else "gemm")]
        assert e["calls"] == 1 and e["bytes"] == 4.0 * (batch * (fin + fout) + 5.0 * fin * fout), (layer, e)


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("widths,batch", [((3, 5, 1), 200), ((201, 135, 35), 200), ((2048, 7, 12), 64), ((2048, 2048, 7), 64),
                                          ((4096, 4096, 3), 4)])
def test_layers_that_begin_between_quads(lib, precision, widths, batch):
    steps_are_equal(lib, widths, batch, precision)
