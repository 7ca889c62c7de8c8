"""Dense weight gradients that update their weights where they are summed up (EpiSgd): the same bits as the gradient and the
update one after the other, at ragged widths, on tiles just filled and batches of a k-tile and its neighbours."""
import numpy as np
import pytest

import synthetic_inputs as S
from gpu_common import build_pair, cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("widths,batch", [((132, 68, 20), 33), ((128, 256, 64), 32), ((264, 72, 1000), 8), ((8, 8, 4), 65),
                                          ((201, 135, 37), 16)])
def test_train_step_equals_gradient_and_update(lib, precision, widths, batch):
    wl = dict(S.MIDI, name="update", fc=list(widths))
    a, b = (build_pair(lib, wl, batch, seed=S.SEED_BASE + 4, pseed=4, std=0.05, bias=0.1, mom_std=0.01, precision=precision)[0]
            for _ in range(2))
    mean = cuda(S.make_mean_image(3, wl["raw"], wl["raw"], S.SEED_BASE + 7))
    for step in range(2):
        raw, labels = (cuda(t) for t in S.make_raw_batch(batch, 3, wl["raw"], wl["raw"], widths[-1], S.SEED_BASE + 40 + step))
        a.preprocess(raw, mean, step, step % 2)
        b.preprocess(raw, mean, step, step % 2)
        la = a.train_step(labels, step, slot=step % 2).cpu()
        lb = b.forward_backward(labels, step, slot=step % 2).cpu()
        b.apply_update()
        assert la.item() == lb.item()
    for pa, pb in ((a.get_params(), b.get_params()), (a.get_momentum(), b.get_momentum())):
        for k in pa:
            assert np.isfinite(pa[k]).all() and np.array_equal(pa[k], pb[k]), k
    a.close()
    b.close()
