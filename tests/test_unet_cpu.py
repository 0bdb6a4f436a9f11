"""Sizes of the network's scratch, host side only: the queried workspace of
every layer and the network's own buffer hold what the smallest call of the
weight gradient with its bias takes (one partial sum per 64 rows)."""
import ctypes

import pytest

from paper_2110_09841_amd import unet as U


def least(ci, co, grid):
    return -(-grid[0] * grid[1] // 64) * (27 * ci * co + co)


# below, at and above 1024 partial sums of the full-resolution layers; rows of a
# quarter of the volume that leave a remainder of 64; the smallest volume
@pytest.mark.parametrize("shape", [(4, 4, 4), (128, 128, 128), (248, 256, 64), (256, 256, 4), (256, 256, 256),
                                   (68, 964, 4), (512, 512, 64)])
def test_workspace_holds_the_weight_and_bias_gradients(shape):
    work = U.work_floats(shape)
    assert work >= 17 * -(-shape[0] * shape[1] * shape[2] // 4096)        # the head's partial sums
    n = ctypes.c_int64()
    for name, ci, co, s in U.LAYERS:
        grid = [v // s for v in shape]
        x, dy = U.NNTensor(None, *grid, ci, ci), U.NNTensor(None, *grid, co, co)
        assert U.lib().cvp_nn_wgrad_workspace(ctypes.byref(x), ctypes.byref(dy), ctypes.byref(n)) == 0
        assert n.value >= least(ci, co, grid), name
        assert work >= n.value, name


def test_workspace_follows_the_volume():
    """No more partial sums than tiles: a small layer asks for little."""
    n = ctypes.c_int64()
    x = U.NNTensor(None, 2, 8, 32, 16, 16)
    assert U.lib().cvp_nn_wgrad_workspace(ctypes.byref(x), ctypes.byref(x), ctypes.byref(n)) == 0
    assert n.value <= 2 * (27 * 16 * 16 + 16)
