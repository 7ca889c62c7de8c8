"""Fused normalisation + pool and its adjoint where their blocks are cut: odd and even maps (last row and column under no window),
one channel quad to 128, windows and exponents other than the network's own, tensors on either side of the line between the
adjoint's two kernels."""
import numpy as np
import pytest

import synthetic_inputs as S
from gpu_common import cuda
from helpers import oracle_spec, rel_l2
from oracle import alexnet_oracle as O

pytestmark = pytest.mark.gpu
OP_RTOL = 2e-5  # as in test_gpu_ops.py: one fp32 operator against float64 on identical inputs


@pytest.mark.parametrize("c,size,n,beta,batch", [
    (4, 6, 5, 0.75, 2), (12, 7, 3, 0.75, 3), (24, 3, 5, 0.75, 1), (96, 9, 5, 0.5, 2), (100, 10, 5, 0.75, 3), (256, 8, 9, 1.0, 2),
    (512, 5, 5, 0.75, 2),
    # large enough for the adjoint on blocks of 2 x 2 pixels; workgroups of unequal shares, lanes without a block
    (96, 9, 5, 0.75, 790), (28, 10, 5, 0.75, 2200), (512, 5, 5, 0.75, 480), (16, 13, 5, 0.75, 6000), (12, 7, 5, 0.75, 28000)])
def test_fused_kernels_at_their_edges(lib, c, size, n, beta, batch):
    wl = dict(S.TINY, crop=size, raw=size, lrn=(n, 2.0, 1e-4, beta),
              conv=[(c, 3, 1, 1, 1, 1, 1)] + [(8, 1, 1, 0, 1, 0, 0)] * 4)
    net = lib.AlexNet(wl, batch)
    spec = oracle_spec(wl, batch)
    a = np.maximum(S.make_normal((batch, c, size, size), 31 + c, std=60.0), 0)
    y, arg = (t.cpu().numpy() for t in net.lrn_pool_forward(1, a))
    b32 = net.lrn_forward(1, a).cpu().numpy()
    want_b, s = O.lrn_forward(a, spec.lrn_n, spec.lrn_k, spec.lrn_alpha, spec.lrn_beta)
    assert rel_l2(b32, want_b) <= OP_RTOL
    want_y, want_arg = O.maxpool_forward(b32, 3, 2)
    assert np.array_equal(y, want_y) and np.array_equal(arg, want_arg)
    dy = S.make_normal(want_y.shape, 57)
    for gate in (True, False):
        da, db = (t.cpu().numpy() for t in net.pool_lrn_backward(1, a, dy, relu_gate=gate))
        want = O.lrn_backward(O.maxpool_backward(dy, want_arg, (size, size)), a, s, spec.lrn_n, spec.lrn_alpha, spec.lrn_beta)
        want = want * (a > 0) if gate else want
        assert rel_l2(da, want) <= OP_RTOL
        assert rel_l2(db, want.sum((0, 2, 3))) <= OP_RTOL * 10  # sums of values of either sign
    net.close()
