"""The autotuner times the kernels that its plan describes, and a stored plan
serves only geometries that keep their records as the timed one did."""
import json

import pytest
import torch

from paper_2110_09841_amd import _lib, autotune as A, cvp, synth

from gpu_util import needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("cached", [False, True])
def test_backprojection_plans_are_timed_without_scratch(cached, monkeypatch):
    G = cvp.Geometry(synth.config_small())
    if cached:
        G.cache_records()
    L, plans = _lib.lib(), []
    call = L.cvp_backproject

    def counted(*args):
        plans.append(G.launch[1:] + (G.bp_workgroups_per_cu, G.bp_shared_window))
        return call(*args)

    monkeypatch.setattr(L, "cvp_backproject", counted)
    rec = A.autotune(G, cvp.Options(variant="relaxed"), bands=(4,), stacks=(16, 8), passes=(2, 1), reps=1)
    say(rec["backproject_ms"])
    assert len(set(plans)) == len(rec["backproject_ms"]) == (16 if cached else 4)


def test_a_stored_plan_serves_the_same_records_only(tmp_path):
    cache = str(tmp_path / "plans.json")
    opts = cvp.Options(variant="relaxed")
    G = cvp.Geometry(synth.config_small())
    few = dict(bands=(4, 8), stacks=(8,), passes=(1,), reps=1, cache=cache)
    assert not A.autotune(G, opts, **few)["cached"]
    assert A.autotune(G, opts, **few)["cached"]
    G.cache_records()
    assert not A.autotune(G, opts, **few)["cached"]
    assert A.autotune(G, opts, **few)["cached"]
    assert len(json.load(open(cache))) == 2
    torch.cuda.synchronize()
