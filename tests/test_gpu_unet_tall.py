"""Network gradients on a slice grid of 256 x 256: the largest number of partial
sums per layer, over a few columns."""
import pytest
import torch

from paper_2110_09841_amd import unet as U

from gpu_util import needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]


def test_gradients_of_a_256_by_256_slice_grid():
    net = U.UNet((256, 256, 4), seed=1)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x1, x2, t = (torch.rand(net.shape, generator=gen, device="cuda") * 0.02 for _ in range(3))
    net.mse(net.forward(x1, x2), t)
    net.backward(net.gx0)
    for name, grad in (("d1a", net.g["d1a"]), ("c3b", net.g["c3b"]), ("c1a", net.g["c1a"])):
        g = grad.double().reshape(-1, grad.shape[3])
        # FP32 sums of fewer than 1000 additions in a row: 1000 * 2^-24 of the absolute sum
        err = (net.convs[name].gb.double() - g.sum(0)).abs()
        say(name, float((err / g.abs().sum(0).clamp(min=1e-300)).max()))
        assert bool((err <= 6e-5 * g.abs().sum(0)).all()), name
        assert bool(torch.isfinite(net.convs[name].gw).all()) and float(net.convs[name].gw.abs().max()) > 0, name
