"""Fixed row counts (a piece of known row count is evaluated without a row
loop), the transposed volume and records made per call: parity with the FP64
oracle for voxels of about 0.6 to 9 detector rows (row counts 2 to 6 and the
general row loop) on detectors that cut the volume off at both row edges, the
same bits for every scratch size (each selects other kernels), and non-finite
projection values reaching only the voxels whose rows they lie on."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from paper_2110_09841_amd import _lib, cvp, synth

from gpu_util import assert_parity, needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]


def geometry(rows_per_voxel, n3, det_rows, cols=58, n_views=5):
    """A 21 x 18 x n3 volume whose slices are about rows_per_voxel detector
    rows high (magnification 1.6), principal row off centre."""
    a3 = rows_per_voxel / 1.6
    return synth.geometry((21, 18, n3), (1.1, 0.9, a3), cols, det_rows, 1.0, 300.0, 480.0, n_views, 200.0,
                          vol_offset_mm=(0.5, -1.0, 0.3 * a3), principal_px=(cols / 2 - 0.7, det_rows / 2 + 1.3))


# (rows per voxel, slices, detector rows): row counts 2, 3, 4, 5, 6 and the
# row loop; slices below, at and above one and two waves of 64, volumes taller
# than the detector and shorter
CASES = [(0.6, 70, 30), (0.9, 129, 141), (1.4, 64, 60), (2.3, 20, 61), (3.4, 9, 25), (4.3, 7, 50), (9.0, 5, 31)]


@pytest.mark.parametrize("variant,ec", [("relaxed", True), ("exact", True), ("relaxed", False), ("exact", False)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%g_rows" % c[0])
def test_row_counts_match_the_oracle(case, variant, ec):
    g = geometry(*case)
    G = cvp.Geometry(g)
    x = synth.uniform_volume(G.vol_shape, seed=5)
    b = synth.uniform_projections(G.proj_shape, seed=6)
    o, opts = O.Options(exact=variant == "exact", ec=ec), cvp.Options(variant=variant, ec=ec)
    say("rows", case, variant, ec, G.launch)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()
    ref_p, ref_b = O.project(g, o, x), O.backproject(g, o, b)
    assert_parity(cvp.project(xd, G, opts).cpu().numpy(), ref_p, "A x")
    back = cvp.backproject(bd, G, opts)
    assert_parity(back.cpu().numpy(), ref_b, "A^T b")
    G.cache_records()
    for gw, kp, wpc, shared in ((16, 2, 4, False), (8, 1, 3, False), (4, 2, 4, False), (8, 2, 4, True), (16, 1, 3, True)):
        G.set_launch(0, gw, kp, wpc, shared)
        assert torch.equal(cvp.backproject(bd, G, opts), back), (gw, kp, wpc, shared)


@pytest.mark.parametrize("variant", ["relaxed", "exact", "tt"])
@pytest.mark.parametrize("rows_per_voxel,n3", [(0.8, 70), (2.3, 21)])
def test_every_scratch_size_gives_the_same_bits(variant, rows_per_voxel, n3):
    g = geometry(rows_per_voxel, n3, 47, n_views=27)
    G = cvp.Geometry(g)
    opts = cvp.TT if variant == "tt" else cvp.Options(variant=variant)
    x = torch.from_numpy(synth.uniform_volume(G.vol_shape, seed=7)).cuda()
    b = torch.from_numpy(synth.uniform_projections(G.proj_shape, seed=8)).cuda()
    p, q = cvp.project(x, G, opts), cvp.backproject(b, G, opts)
    o, L = opts.c(), _lib.lib()
    full = ctypes.c_int64(), ctypes.c_int64()
    _lib.check(L.cvp_operator_workspace_size(G.handle, ctypes.byref(o), ctypes.byref(full[0]), ctypes.byref(full[1])))
    per_view = 21 * 18 * 4 * (4 * 12 + 1)
    vt = 4 * x.numel() + 512 + 4 * G.project_work_words
    sums = 4 * 2 * 4 * 2 * 64 * 18 * 32 * ((n3 + 63) // 64)       # bounds the running sums of any stack shape
    ptr = ctypes.c_void_p

    def run(nbytes, shift):
        work = torch.full((nbytes + shift,), 0x7f, dtype=torch.uint8, device="cuda")    # NaN-like bytes
        po, qo = torch.full_like(p, float("nan")), torch.full_like(q, float("nan"))
        w = ptr(work.data_ptr() + shift)
        say("scratch", variant, rows_per_voxel, nbytes, shift)
        if nbytes >= 4 * G.project_work_words:
            _lib.check(L.cvp_project_ws(G.handle, ctypes.byref(o), ptr(x.data_ptr()), ptr(po.data_ptr()), w, nbytes,
                                        cvp._stream()))
            assert torch.equal(po, p), nbytes
        _lib.check(L.cvp_backproject_ws(G.handle, ctypes.byref(o), ptr(b.data_ptr()), ptr(qo.data_ptr()), w, nbytes,
                                        cvp._stream()))
        assert torch.equal(qo, q), nbytes

    for nbytes in (0, 4 * G.project_work_words, vt, vt + 9 * per_view, sums + 13 * per_view, max(f.value for f in full)):
        for shift in (0, 4):
            run(nbytes, shift)
    run(vt + 27 * per_view + 4096, 16)


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("rows_per_voxel,n3", [(0.8, 70), (2.3, 21)])
def test_non_finite_projection_values_stay_local(rows_per_voxel, n3, cached):
    """An infinite pixel: every voxel with weight on it is non-finite, and none
    that has no weight on its row or the next ones (the row loop's range
    reaches at most one row further than the weights)."""
    g = geometry(rows_per_voxel, n3, 61)
    G = cvp.Geometry(g)
    if cached:
        G.cache_records()
    b = synth.uniform_projections(G.proj_shape, seed=9)
    view, v, u = 2, 30, 29
    o = O.Options(exact=False, ec=True)
    one, wide = np.zeros(b.shape), np.zeros(b.shape)
    one[view, v, u] = 1.0
    wide[view, v - 1:v + 2, u] = 1.0
    reach, near = O.backproject(g, o, one) > 0, O.backproject(g, o, wide) > 0
    b[view, v, u] = np.inf
    got = cvp.backproject(torch.from_numpy(b).cuda(), G, cvp.Options(variant="relaxed")).cpu().numpy()
    bad = ~np.isfinite(got)
    say("non-finite", rows_per_voxel, int(reach.sum()), int(bad.sum()), int(near.sum()))
    assert reach.any() and not (reach & ~bad).any() and not (bad & ~near).any()
    b[view, v, u] = 0.0
    ref = O.backproject(g, o, b)
    assert_parity(got[~near], ref[~near], "voxels beside the infinite pixel")
