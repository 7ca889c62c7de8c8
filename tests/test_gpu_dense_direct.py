"""Dense layers of bf16 handles in whole steps (csrc/weight_direct.hip, gemm_direct.h): widths that are multiples of eight but of
no tile and no k-tile, 64- and 128-row tiles that end inside the batch, reductions in one and in many slices."""
import pytest

import synthetic_inputs as S
from gpu_common import BF16_OWN_DECISIONS_RTOL, run_step_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,batch", [([2056, 1032, 504], 70), ([2056, 1032, 504], 37), ([4104, 2056, 200], 130)])
def test_steps_with_wide_dense_layers(lib, widths, batch):
    """The bars of the other bf16 steps (tests/test_gpu_bf16.py)."""
    wl = dict(S.MINI)
    wl["name"] = "mini_wide"
    wl["fc"] = widths
    run_step_and_compare(lib, wl, batch, seed=21, bias=0.1, std=0.03, use_raw=False, steps=1, mom_std=0.01, precision=1,
                         direct=True, direct_tol=BF16_OWN_DECISIONS_RTOL, direct_report={}, loss_rtol=1e-2, tol=2e-2,
                         report={})
