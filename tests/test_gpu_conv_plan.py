"""Convolutions of tall, narrow volumes: planning the march stays short on the
host however many slices there are, and the results are exact."""
import ctypes
import time

import pytest
import torch

from paper_2110_09841_amd import unet as U

from gpu_util import say
from test_gpu_conv_edges import ints, reference

pytestmark = pytest.mark.gpu


def test_planning_a_tall_volume_takes_little_host_time():
    x, w = ints((200000, 1, 1, 16), 1), ints((27, 16, 16), 2)
    y = torch.empty_like(x)
    dw, n = torch.empty((27, 16, 16), device="cuda"), ctypes.c_int64()
    xd, yd, L = U.desc(x), U.desc(y), U.lib()
    U._check(L.cvp_nn_wgrad_workspace(ctypes.byref(xd), ctypes.byref(yd), ctypes.byref(n)))
    work = torch.empty(n.value, device="cuda")
    conv = lambda: L.cvp_nn_conv3d(ctypes.byref(xd), U._p(w), None, ctypes.byref(yd), 0, 0, U._s())
    wgrad = lambda: L.cvp_nn_conv3d_wgrad(ctypes.byref(xd), ctypes.byref(yd), U._p(dw), U._p(work), n.value, U._s())
    for call in (conv, wgrad):
        times = []
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            U._check(call())
            times.append(time.perf_counter() - t)
        say("host time of a call on 200000 slices: %.0f us" % (1e6 * min(times)))
        assert min(times) < 5e-4
    taps = [9 * d + 4 for d in range(3)]                  # the others meet the padding
    xp = torch.zeros((200002, 16), dtype=torch.float64)
    xp[1:-1] = x[:, 0, 0].double().cpu()
    ref = sum(xp[d:d + 200000] @ w[taps[d]].double().cpu().t() for d in range(3))
    assert torch.equal(y[:, 0, 0].cpu(), ref.float().to(torch.bfloat16))


@pytest.mark.parametrize("shape", [(700, 3, 5), (1025, 1, 33)])
def test_tall_volumes_are_exact(shape):
    x, g = ints(shape + (16,), 3), ints(shape + (32,), 4)
    dw, n = torch.empty((27, 32, 16), device="cuda"), ctypes.c_int64()
    xd, gd, L = U.desc(x), U.desc(g), U.lib()
    U._check(L.cvp_nn_wgrad_workspace(ctypes.byref(xd), ctypes.byref(gd), ctypes.byref(n)))
    work = torch.full((n.value,), float("nan"), device="cuda")
    U._check(L.cvp_nn_conv3d_wgrad(ctypes.byref(xd), ctypes.byref(gd), U._p(dw), U._p(work), n.value, U._s()))
    assert torch.equal(dw.cpu(), reference(x, g))
