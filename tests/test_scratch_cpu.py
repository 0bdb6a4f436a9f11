"""Scratch of the operators, host side: what a geometry's bound leaves of it,
and allocations outside torch that find the memory in torch's cache."""
import pytest
import torch

from paper_2110_09841_amd import _lib, cvp


class Geom:
    handle = None
    project_work_words = 100
    scratch_bytes = None


class FakeLib:
    def cvp_operator_workspace_size(self, g, o, p, b):
        p._obj.value, b._obj.value = 1000000, 3000000
        return _lib.CVP_OK


@pytest.mark.parametrize("bound,project,back,both", [(None, 1000000, 3000000, 3000000), (5000000, 1000000, 3000000, 3000000),
                                                     (2000000, 1000000, 2000000, 2000000), (1000, 1000, 1000, 1000),
                                                     (300, 400, 300, 400), (0, 400, 0, 400)])
def test_the_bound_of_a_geometry(bound, project, back, both, monkeypatch):
    monkeypatch.setattr(_lib, "lib", FakeLib)
    g, o = Geom(), _lib.OptionsC()
    g.scratch_bytes = bound
    size = lambda **kw: cvp.operator_scratch(g, o, "cpu", **kw).numel()
    assert size(backproject=False) == project and size(project=False) == back and size() == both


def test_a_second_try_without_torchs_unused_memory(monkeypatch):
    freed = []
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: freed.append(1))
    tries = [_lib.CVP_E_NOMEM, _lib.CVP_OK]
    cvp._with_freed_cache(lambda: tries.pop(0))
    assert freed == [1] and tries == []
    for first, again in ((_lib.CVP_E_NOMEM, 2), (_lib.CVP_E_UNSUPPORTED, 1), (_lib.CVP_E_DEVICE, 1)):
        calls = []
        with pytest.raises(_lib.CVPError):
            cvp._with_freed_cache(lambda: calls.append(1) or first)
        assert len(calls) == again


def test_geometries_are_unbounded_by_default():
    assert cvp.Geometry.scratch_bytes is None
