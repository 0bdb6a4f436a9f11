"""Operators and solvers of a geometry with bounded scratch: the results of the
unbounded ones, within the bound."""
import pytest
import torch

from paper_2110_09841_amd import autograd, cvp, solvers, synth

from gpu_util import needs_gpu, say
from test_gpu_records import geoms

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("name", ["pmax4", "pmax8"])
def test_bounded_scratch_gives_the_same_bits(name):
    g = geoms()[name]
    opts = cvp.Options(variant="relaxed")

    def run(G):
        x = torch.from_numpy(synth.uniform_volume(G.vol_shape, seed=51)).cuda().requires_grad_()
        b = torch.from_numpy(synth.uniform_projections(G.proj_shape, seed=52)).cuda()
        p = autograd.project(x, G, opts)
        (p * b).sum().backward()
        out = [p.detach(), x.grad, solvers.backproject_views(b, G, 1, 3, 3, opts=opts)]
        for S, n in ((cvp.CGLS(G, opts, b), 3), (solvers.LSQR(G, opts, b), 3)):
            S.start()
            S.iterate(n)
            out.append(S.x)
        S = solvers.OSSART(G, opts, b, 3)
        S.setup()
        S.iterate(2)
        return out + [S.x], S.scratch.numel()

    ref, full = run(cvp.Geometry(g))
    for bound in (0, 4096, full // 3, full):
        G = cvp.Geometry(g)
        G.scratch_bytes = bound
        got, used = run(G)
        say(name, "scratch bound", bound, "of", full, "taken", used)
        assert used <= max(bound, 4 * G.project_work_words)
        for a, r in zip(got, ref):
            assert torch.equal(a, r), bound
