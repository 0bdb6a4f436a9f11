"""The 3x3x3 convolution and its weight gradient: tile edges, channel pairs,
workspace sizes.  The inputs are small whole numbers, whose products and sums
FP32 holds exactly, so the results are compared for equality."""
import ctypes

import pytest
import torch

from paper_2110_09841_amd import unet as U

pytestmark = pytest.mark.gpu


def wgrad(x, g, floats=None):
    L = U.lib()
    n = ctypes.c_int64()
    xd, gd = U.desc(x), U.desc(g)
    U._check(L.cvp_nn_wgrad_workspace(ctypes.byref(xd), ctypes.byref(gd), ctypes.byref(n)))
    floats = n.value if floats is None else floats
    assert floats <= n.value
    work = torch.full((floats,), float("nan"), device="cuda")
    dw = torch.empty((27, g.shape[3], x.shape[3]), device="cuda")
    st = L.cvp_nn_conv3d_wgrad(ctypes.byref(xd), ctypes.byref(gd), U._p(dw), U._p(work), floats, U._s())
    return st, dw


def reference(x, g):
    x, g = x.double().cpu(), g.double().cpu()
    D, H, W, ci = x.shape
    xp = torch.zeros(D + 2, H + 2, W + 2, ci, dtype=torch.float64)
    xp[1:-1, 1:-1, 1:-1] = x
    gm = g.reshape(-1, g.shape[3]).t()
    return torch.stack([gm @ xp[t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, ci)
                        for t in range(27)]).float()


def ints(shape, seed):
    gen = torch.Generator().manual_seed(seed)
    return torch.randint(-4, 5, shape, generator=gen).to(torch.bfloat16).cuda()


@pytest.mark.parametrize("co,ci", [(16, 16), (16, 32), (16, 64), (32, 16), (32, 32), (32, 64), (64, 32), (64, 64)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 9, 16), (5, 17, 33), (2, 8, 66), (70, 5, 31)])
def test_weight_gradient_is_exact_for_whole_numbers(co, ci, shape):
    x, g = ints(shape + (ci,), 1), ints(shape + (co,), 2)
    st, dw = wgrad(x, g)
    assert st == 0
    assert torch.equal(dw.cpu(), reference(x, g))


@pytest.mark.parametrize("co,ci", [(16, 16), (64, 64)])
def test_weight_gradient_with_the_smallest_workspace(co, ci):
    x, g = ints((40, 7, 70, ci), 3), ints((40, 7, 70, co), 4)
    least = (40 * 7 + 63) // 64 * 27 * co * ci
    st, dw = wgrad(x, g, least)
    assert st == 0 and torch.equal(dw.cpu(), reference(x, g))
    assert wgrad(x, g, least - 1)[0] != 0


def test_infinite_input_at_the_row_end_meets_no_padding():
    """An infinite X in the last voxel of a row makes exactly those taps
    non-finite that pair it with a voxel of the gradient."""
    x, g = ints((1, 1, 20, 16), 5), torch.ones((1, 1, 20, 16), dtype=torch.bfloat16, device="cuda")
    x[0, 0, 19, 3] = float("inf")
    st, dw = wgrad(x, g)
    assert st == 0
    bad = ~torch.isfinite(dw[12:15].cpu())          # dz = dy = 0, dx = -1, 0, 1
    want = torch.zeros_like(bad)
    want[1:, :, 3] = True                           # dY at 19 (dx = 0) and at 18 (dx = 1)
    assert torch.equal(bad, want)


@pytest.mark.parametrize("co", [16, 32, 64])
@pytest.mark.parametrize("ci", [16, 32, 64])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 9, 16), (5, 17, 33), (2, 8, 66), (70, 5, 31)])
@pytest.mark.parametrize("flip", [0, 1])
def test_convolution_is_exact_for_whole_numbers(co, ci, shape, flip):
    """Input and output are channel slices; the channels beside the output
    keep their values."""
    D, H, W = shape
    x, w = ints(shape + (ci + 8,), 6), ints((27, co, ci), 7)
    bias = None if flip else ints((co,), 8).float()
    y = torch.full(shape + (co + 24,), 3.0, dtype=torch.bfloat16, device="cuda")
    U._check(U.lib().cvp_nn_conv3d(ctypes.byref(U.desc(x, 8, ci)), U._p(w), U._p(bias), ctypes.byref(U.desc(y, 16, co)),
                                   1 - flip, flip, U._s()))
    xp = torch.zeros(D + 2, H + 2, W + 2, ci, dtype=torch.float64)
    xp[1:-1, 1:-1, 1:-1] = x[..., 8:].double().cpu()
    ref = torch.zeros(D, H, W, co, dtype=torch.float64)
    for t in range(27):
        m = 26 - t if flip else t
        ref += xp[m // 9:m // 9 + D, m // 3 % 3:m // 3 % 3 + H, m % 3:m % 3 + W] @ w[t].double().cpu().t()
    if not flip:
        ref = (ref + bias.double().cpu()).clamp(min=0)
    y = y.cpu()
    assert torch.equal(y[..., 16:16 + co], ref.float().to(torch.bfloat16))
    assert (y[..., :16] == 3).all() and (y[..., 16 + co:] == 3).all()


@pytest.mark.parametrize("flip", [0, 1])
def test_infinite_weight_and_input_stay_local(flip):
    """16 input channels: the last k step holds one tap; an infinite voxel
    reaches its 27 neighbours and no others."""
    x = torch.ones((5, 6, 40, 16), dtype=torch.bfloat16, device="cuda")
    x[2, 3, 20, 5] = float("inf")
    w = torch.ones((27, 16, 16), dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(x)
    U._check(U.lib().cvp_nn_conv3d(ctypes.byref(U.desc(x)), U._p(w), None, ctypes.byref(U.desc(y)), 0, flip, U._s()))
    bad = ~torch.isfinite(y.cpu())
    want = torch.zeros_like(bad)
    want[1:4, 2:5, 19:22] = True
    assert torch.equal(bad, want)


def same_bits(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("ci,co", [(16, 16), (16, 32), (32, 16), (32, 32), (32, 64), (64, 32), (64, 64), (24, 16)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 17, 33), (2, 8, 66)])
def test_masked_backward_equals_convolution_and_mask(ci, co, shape):
    L, gen = U.lib(), torch.Generator().manual_seed(9)
    dy = torch.randn(shape + (ci,), generator=gen).to(torch.bfloat16).cuda()
    w = torch.randn((27, co, ci), generator=gen).to(torch.bfloat16).cuda()
    keep = torch.randn(shape + (co + 8,), generator=gen).clamp(min=0).to(torch.bfloat16).cuda()
    a, b = (torch.full(shape + (co + 8,), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    k = U.desc(keep, 0, co)
    U._check(L.cvp_nn_conv3d(ctypes.byref(U.desc(dy)), U._p(w), None, ctypes.byref(U.desc(a, 8, co)), 0, 1, U._s()))
    U._check(L.cvp_nn_relu_mask(ctypes.byref(U.desc(a, 8, co)), ctypes.byref(k), U._s()))
    U._check(L.cvp_nn_conv3d_bwd_masked(ctypes.byref(U.desc(dy)), U._p(w), ctypes.byref(k),
                                        ctypes.byref(U.desc(b, 8, co)), U._s()))
    assert same_bits(a, b)


@pytest.mark.parametrize("co,ci", [(16, 16), (32, 64), (64, 32)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 17, 33), (70, 5, 31)])
def test_bias_gradient_beside_the_weights(co, ci, shape):
    L = U.lib()
    x, g = ints(shape + (ci,), 1), ints(shape + (co,), 2)
    dw, db = torch.empty((27, co, ci), device="cuda"), torch.empty(co, device="cuda")
    least = (shape[0] * shape[1] + 63) // 64 * (27 * co * ci + co)
    for floats in (least, 20 * least):
        work = torch.full((floats,), float("nan"), device="cuda")
        U._check(L.cvp_nn_conv3d_wgrad_bias(ctypes.byref(U.desc(x)), ctypes.byref(U.desc(g)), U._p(dw), U._p(db),
                                            U._p(work), floats, U._s()))
        assert torch.equal(dw.cpu(), reference(x, g))
        assert torch.equal(db.cpu(), g.float().sum((0, 1, 2)).cpu())


def test_masked_upsampling_pooling_and_head():
    L, gen = U.lib(), torch.Generator().manual_seed(10)
    rnd = lambda s: torch.randn(s, generator=gen).to(torch.bfloat16).cuda()
    fine, coarse = (6, 4, 10), (3, 2, 5)
    gf, kc = rnd(fine + (16,)), rnd(coarse + (16,)).clamp(min=0)
    a, b = torch.empty_like(kc), torch.empty_like(kc)
    U._check(L.cvp_nn_upsample2_bwd(ctypes.byref(U.desc(gf)), ctypes.byref(U.desc(a)), U._s()))
    U._check(L.cvp_nn_relu_mask(ctypes.byref(U.desc(a)), ctypes.byref(U.desc(kc)), U._s()))
    U._check(L.cvp_nn_upsample2_bwd_masked(ctypes.byref(U.desc(gf)), ctypes.byref(U.desc(kc)), ctypes.byref(U.desc(b)),
                                           U._s()))
    assert same_bits(a, b)
    gc, kf = rnd(coarse + (16,)), rnd(fine + (16,)).clamp(min=0)
    a, b, t = gf.clone(), gf.clone(), torch.empty_like(gf)
    U._check(L.cvp_nn_avgpool2_bwd(ctypes.byref(U.desc(gc)), ctypes.byref(U.desc(t)), U._s()))
    U._check(L.cvp_nn_add(ctypes.byref(U.desc(a)), ctypes.byref(U.desc(t)), ctypes.byref(U.desc(a)), U._s()))
    U._check(L.cvp_nn_relu_mask(ctypes.byref(U.desc(a)), ctypes.byref(U.desc(kf)), U._s()))
    U._check(L.cvp_nn_avgpool2_bwd_add(ctypes.byref(U.desc(gc)), ctypes.byref(U.desc(kf)), ctypes.byref(U.desc(b)), U._s()))
    assert same_bits(a, b)
    w, gx = torch.randn(16, generator=gen).cuda(), torch.randn(fine, generator=gen).cuda()
    work = torch.empty(4096, device="cuda")
    d1, d2 = torch.empty(17, device="cuda"), torch.empty(17, device="cuda")
    U._check(L.cvp_nn_head_bwd(ctypes.byref(U.desc(kf)), U._p(w), U._p(gx), ctypes.c_float(2.0), ctypes.byref(U.desc(a)),
                               U._p(d1), U._p(work), 4096, U._s()))
    U._check(L.cvp_nn_relu_mask(ctypes.byref(U.desc(a)), ctypes.byref(U.desc(kf)), U._s()))
    U._check(L.cvp_nn_head_bwd_masked(ctypes.byref(U.desc(kf)), U._p(w), U._p(gx), ctypes.c_float(2.0),
                                      ctypes.byref(U.desc(b)), U._p(d2), U._p(work), 4096, U._s()))
    assert same_bits(a, b) and torch.equal(d1, d2)
