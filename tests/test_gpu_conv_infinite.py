"""An infinite weight of a 3x3x3 convolution: infinite results of its output
channel where its tap meets the volume, NaN where it meets the zero padding,
and no other channel touched."""
import ctypes

import pytest
import torch

from paper_2110_09841_amd import unet as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flip", [0, 1])
@pytest.mark.parametrize("tap", [0, 12, 26])        # 26: alone in the last k step with 16 input channels
@pytest.mark.parametrize("ci,co", [(16, 16), (32, 16), (64, 32), (24, 16)])
def test_infinite_weight_stays_in_its_channel_and_tap(ci, co, tap, flip):
    D, H, W = 3, 5, 35
    x = torch.ones((D, H, W, ci), dtype=torch.bfloat16, device="cuda")
    w = torch.ones((27, co, ci), dtype=torch.bfloat16, device="cuda")
    w[tap, 3, 5] = float("inf")
    y = torch.empty((D, H, W, co), dtype=torch.bfloat16, device="cuda")
    U._check(U.lib().cvp_nn_conv3d(ctypes.byref(U.desc(x)), U._p(w), None, ctypes.byref(U.desc(y)), 0, flip, U._s()))
    m = 26 - tap if flip else tap
    inside = torch.zeros((D + 2, H + 2, W + 2), dtype=torch.bool)
    inside[1:-1, 1:-1, 1:-1] = True
    inside = inside[m // 9:m // 9 + D, m // 3 % 3:m // 3 % 3 + H, m % 3:m % 3 + W]
    y = y.float().cpu()
    assert torch.equal(y[..., 3] == float("inf"), inside) and torch.equal(torch.isnan(y[..., 3]), ~inside)
    assert torch.isfinite(y[..., [c for c in range(co) if c != 3]]).all()
