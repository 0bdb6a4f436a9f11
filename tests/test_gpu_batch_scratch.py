"""The scratch of a batch: bounded by what its creator allows, filled by every
call, and without effect on the results -- members with and without cached
records, 4 and 8 pieces per column, every stack width of the kernels that a
batch without room for copies runs."""
import pytest
import torch

from paper_2110_09841_amd import _lib, cvp, synth

from gpu_util import needs_gpu, say
from test_gpu_records import COMBOS, geoms

pytestmark = [pytest.mark.gpu, needs_gpu]


def members():
    """Stack widths 16, 8 and 4 with 4 pieces, 8 and 4 with 8 pieces (wider
    ones do not fit)."""
    gs = geoms()
    out = []
    for name, gw in (("pmax4", 16), ("pmax4", 8), ("pmax4", 4), ("pmax8", 8), ("pmax8", 4)):
        out.append(cvp.Geometry(gs[name]))
        out[-1].set_launch(0, gw, 2 if gw == 4 else 1)
    return out


def sizes(G):
    """Bytes of the members' records, and of the larger kind of copies."""
    rec = sum(g.n_views * g.vol_shape[1] * g.vol_shape[2] * 8 * (4 * 12 + 1) * 4 for g in G)
    copies = sum(max(4 * g.n_voxels, g.n_views * g.proj_shape[2] * 4 * (g.proj_shape[1] + 12) + 4096) for g in G)
    return rec, copies


@pytest.mark.parametrize("keep", ["none", "some", "all"])
def test_results_do_not_depend_on_the_scratch(keep):
    G = members()
    for g in G[::2] if keep == "some" else G if keep == "all" else []:
        g.cache_records()
    xs = [torch.from_numpy(synth.uniform_volume(g.vol_shape, seed=31 + q)).cuda() for q, g in enumerate(G)]
    bs = [torch.from_numpy(synth.uniform_projections(g.proj_shape, seed=41 + q)).cuda() for q, g in enumerate(G)]
    refs = {c: ([cvp.project(x, g, cvp.Options(variant=c[0], ec=c[1])) for x, g in zip(xs, G)],
                [cvp.backproject(b, g, cvp.Options(variant=c[0], ec=c[1])) for b, g in zip(bs, G)]) for c in COMBOS}
    rec, copies = sizes(G)
    for limit in (0, 4096, rec // 16, rec, copies, rec + copies + (1 << 20), None):
        batch = cvp.Batch(G, limit)
        say("batch scratch", keep, limit)
        for c in COMBOS:
            opts = cvp.Options(variant=c[0], ec=c[1])
            for rep in range(2):
                ps = [torch.full(g.proj_shape, float("nan"), device="cuda") for g in G]
                vs = [torch.full(g.vol_shape, float("nan"), device="cuda") for g in G]
                cvp.project_batched(xs, batch, opts, outs=ps)
                cvp.backproject_batched(bs, batch, opts, outs=vs)
                for q in range(len(G)):
                    assert torch.equal(ps[q], refs[c][0][q]), (limit, c, q)
                    assert torch.equal(vs[q], refs[c][1][q]), (limit, c, q)


def test_the_bound_holds():
    """Device memory that a batch takes (allocations come in steps of 2 MiB)."""
    g = synth.geometry((96, 96, 96), 1.0, 160, 140, 1.6, 300.0, 520.0, 60, 360.0)
    G = [cvp.Geometry(g) for _ in range(2)]
    torch.cuda.synchronize()
    for limit in (0, 1 << 20, 64 << 20):
        free = torch.cuda.mem_get_info()[0]
        batch = cvp.Batch(G, limit)
        used = free - torch.cuda.mem_get_info()[0]
        say("batch of 2 x 96^3 x 60 views, scratch", limit, "takes", used)
        assert used <= limit + (16 << 20)
        del batch


def test_a_negative_bound_is_refused():
    with pytest.raises(_lib.CVPError) as ei:
        cvp.Batch([cvp.Geometry(geoms()["pmax4"])], -1)
    assert ei.value.status == _lib.CVP_E_INVALID
