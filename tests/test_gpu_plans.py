"""Backprojections without scratch, whose kernels stage detector windows and
follow the launch plan: every stack, pass count, LDS budget and window form,
with and without a table of records, gives the bits of the launch with scratch
(which reads a transposed copy and ignores those fields), for row counts 2 to 6
and the row loop, 4 and 8 pieces per column, windows in LDS and windows too
large for it, and with infinite pixels."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from paper_2110_09841_amd import _lib, cvp, synth

from gpu_util import assert_parity, needs_gpu, say
from test_gpu_fixed_rows import CASES, geometry
from test_gpu_records import COMBOS, geoms

pytestmark = [pytest.mark.gpu, needs_gpu]

# (stack columns, passes, workgroups per CU, one window per workgroup)
UNCACHED = [(gw, kp, 0, False) for gw in (16, 8, 4) for kp in (2, 1)]
CACHED = [(16, 2, 4, False), (8, 1, 3, False), (4, 2, 4, False), (4, 1, 3, False), (8, 2, 4, True), (16, 1, 3, True),
          (16, 2, 3, True)]


def back(b, G, opts, views=None):
    """x = A^T b by the entry points without scratch (views: first, step, count)."""
    out = torch.full(G.vol_shape, float("nan"), device="cuda")
    o, L = opts.c(), _lib.lib()
    args = G.handle, ctypes.byref(o), ctypes.c_void_p(b.data_ptr()), ctypes.c_void_p(out.data_ptr())
    _lib.check(L.cvp_backproject(*args, cvp._stream()) if views is None else
               L.cvp_backproject_views(*args, *views, cvp._stream()))
    return out


def plans(G, cached):
    """Sets the plans that fit, one after another."""
    set_any = 0
    for gw, kp, wpc, shared in CACHED if cached else UNCACHED:
        try:
            G.set_launch(0, gw, kp, wpc, shared)
        except _lib.CVPError as e:
            assert e.status == _lib.CVP_E_UNSUPPORTED
            continue
        assert G.bp_shared_window == shared and G.launch[1:] == (gw, kp)
        set_any += 1
        yield gw, kp, wpc, shared
    assert set_any >= 4


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%g_rows" % c[0])
def test_every_plan_gives_the_bits_of_the_launch_with_scratch(case, cached):
    g = geometry(*case)
    G = cvp.Geometry(g)
    b = torch.from_numpy(synth.uniform_projections(G.proj_shape, seed=11)).cuda()
    forms = [cvp.Options(variant=v, ec=ec) for v, ec in COMBOS] + ([] if cached else [cvp.TT])
    ref = [cvp.backproject(b, G, o) for o in forms]
    if cached:
        G.cache_records()
    for plan in plans(G, cached):
        say("plan", case, cached, plan)
        for o, r in zip(forms, ref):
            assert torch.equal(back(b, G, o), r), (plan, o)


@pytest.mark.parametrize("cached", [False, True])
def test_eight_pieces_and_windows_beyond_the_lds(cached):
    """Pixels small against the voxels: the windows of the wide stacks are read
    from the caller's projections; view subsets; parity with the oracle."""
    g = geoms()["pmax8"]
    G = cvp.Geometry(g)
    b = synth.uniform_projections(G.proj_shape, seed=12)
    refs = {(v, ec): O.backproject(g, O.Options(exact=v == "exact", ec=ec), b) for v, ec in COMBOS}
    b = torch.from_numpy(b).cuda()
    if cached:
        G.cache_records()
    subset = None
    for plan in plans(G, cached):
        say("eight pieces", cached, plan)
        for v, ec in COMBOS:
            o = cvp.Options(variant=v, ec=ec)
            got = back(b, G, o)
            assert torch.equal(got, cvp.backproject(b, G, o)), (plan, v, ec)
        assert_parity(got.cpu().numpy(), refs[v, ec], "A^T b, no scratch, %s" % (plan,))
        part = back(b, G, o, (1, 3, 3))
        assert subset is None or torch.equal(part, subset), plan
        subset = part


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("name", ["0.8_rows", "2.3_rows", "pmax8"])
def test_infinite_pixels_stay_local_under_every_plan(name, cached):
    """An infinite pixel reaches every voxel with weight on it and none without
    weight on its row or the next ones."""
    g = geoms()["pmax8"] if name == "pmax8" else geometry(*{"0.8_rows": (0.8, 70, 61), "2.3_rows": (2.3, 21, 61)}[name])
    G = cvp.Geometry(g)
    if cached:
        G.cache_records()
    b = synth.uniform_projections(G.proj_shape, seed=13)
    view, v, u = 2, G.proj_shape[1] // 2, G.proj_shape[2] // 2
    o = O.Options(exact=False, ec=True)
    one, wide = np.zeros(b.shape), np.zeros(b.shape)
    one[view, v, u] = 1.0
    wide[view, v - 1:v + 2, u] = 1.0
    reach, near = O.backproject(g, o, one) > 0, O.backproject(g, o, wide) > 0
    b[view, v, u] = np.inf
    d = torch.from_numpy(b).cuda()
    b[view, v, u] = 0.0
    ref = O.backproject(g, o, b)
    assert reach.any()
    for plan in plans(G, cached):
        say("infinite pixel", name, cached, plan)
        got = back(d, G, cvp.Options(variant="relaxed")).cpu().numpy()
        bad = ~np.isfinite(got)
        assert not (reach & ~bad).any() and not (bad & ~near).any(), plan
        assert_parity(got[~near], ref[~near], "voxels beside the infinite pixel")
