"""Projections on the caller's layout (no scratch, the group maxima alone, or
few slices): one and two slices per lane, with and without a table of records,
give the bits of the launch with scratch."""
import ctypes

import pytest
import torch

from paper_2110_09841_amd import _lib, cvp, synth

from gpu_util import needs_gpu, say
from test_gpu_fixed_rows import CASES, geometry
from test_gpu_records import COMBOS, geoms

pytestmark = [pytest.mark.gpu, needs_gpu]


def project(x, G, opts, entry, work=()):
    out = torch.full(G.proj_shape, float("nan"), device="cuda")
    o = opts.c()
    _lib.check(getattr(_lib.lib(), entry)(G.handle, ctypes.byref(o), ctypes.c_void_p(x.data_ptr()),
                                          ctypes.c_void_p(out.data_ptr()), *work, cvp._stream()))
    return out


# slices: 5 to 129 of CASES, and 65, 128, 192, 193 (second slices partly or wholly
# beyond the volume, several rounds), bands of 1 and 3 columns and the default
@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("case", CASES + [(0.7, 65, 33), (0.6, 128, 50), (0.5, 192, 70), (0.5, 193, 40), "pmax8"],
                         ids=lambda c: c if isinstance(c, str) else "%g_rows_%d" % c[:2])
def test_projection_without_scratch(case, cached):
    G = cvp.Geometry(geoms()[case] if isinstance(case, str) else geometry(*case))
    x = torch.from_numpy(synth.uniform_volume(G.vol_shape, seed=21)).cuda()
    if cached:
        G.cache_records()
    least = torch.empty(G.project_work_words, dtype=torch.int32, device="cuda")
    forms = [cvp.Options(variant=v, ec=ec) for v, ec in COMBOS] + [cvp.TT]
    for u in (0, 1, 3):
        G.set_launch(u)
        say("no scratch", case, cached, G.launch)
        for o in forms:
            ref = cvp.project(x, G, o)
            assert torch.isfinite(ref).all()
            assert torch.equal(project(x, G, o, "cvp_project"), ref), (u, o)
            assert torch.equal(project(x, G, o, "cvp_project_noalloc"), ref), (u, o)
            work = ctypes.c_void_p(least.data_ptr()), 4 * least.numel()
            assert torch.equal(project(x, G, o, "cvp_project_ws", work), ref), (u, o)
