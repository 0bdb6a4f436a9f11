"""Volumes of so many columns that the narrow stacks of the backprojection from
transposed projections exceed the threads of a launch: the call with scratch
takes the kernels without a copy."""
import ctypes

import pytest
import torch

from paper_2110_09841_amd import _lib, cvp, synth

from gpu_util import needs_gpu, say
from test_gpu_plans import back

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("edge", [8180, 8192])
def test_backprojection_of_a_wide_slice(edge):
    g = synth.geometry((edge, edge, 1), 0.05, 300, 9, 5.0, 750.0, 1200.0, 1, 360.0)
    G = cvp.Geometry(g)
    opts = cvp.Options(variant="relaxed")
    b = torch.from_numpy(synth.uniform_projections(G.proj_shape, seed=61)).cuda()
    p, q, o = ctypes.c_int64(), ctypes.c_int64(), opts.c()
    _lib.check(_lib.lib().cvp_operator_workspace_size(G.handle, ctypes.byref(o), ctypes.byref(p), ctypes.byref(q)))
    say("columns", edge * edge, "scratch", q.value)
    assert (q.value == 0) == (edge == 8192)
    got = cvp.backproject(b, G, opts)
    assert torch.equal(got, back(b, G, opts)) and bool(torch.isfinite(got).all()) and float(got.max()) > 0
    # any scratch is taken
    work = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    out = torch.full_like(got, float("nan"))
    _lib.check(_lib.lib().cvp_backproject_ws(G.handle, ctypes.byref(o), ctypes.c_void_p(b.data_ptr()),
                                             ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(work.data_ptr()),
                                             work.numel(), cvp._stream()))
    assert torch.equal(out, got)
