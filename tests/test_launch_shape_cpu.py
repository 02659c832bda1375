"""The launch shape that the batched call's binding hands to the library: a
launch mode that the caller names is kept, also mode 0 (the persistent launch),
whose number is that of a field left alone."""
import copy

import pytest

from paper_2204_04898_amd import pm4g, tune


@pytest.fixture(params=[None, {"tile_events": 2048, "emit_blocks": 77, "agg_blocks": 99, "launch": 1},
                        {"tile_events": 2048, "emit_blocks": 77, "agg_blocks": 99, "launch": 0}])
def hit(request, monkeypatch):
    class Fixed:
        def lookup(self, *a):
            return dict(request.param) if request.param is not None else None
    monkeypatch.setattr(tune, "default_cache", lambda: Fixed())
    return request.param


def _shape(tuning):
    t = pm4g._launch_shape(tuning, 20, 5, 1000)
    return t.tile_events, t.emit_blocks, t.agg_blocks, t.launch


def _assigned(v):
    t = pm4g.BatchedTuning(pair_capacity=7)
    t.launch = v
    return t


@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("make", [lambda v: pm4g.BatchedTuning(launch=v), lambda v: pm4g.BatchedTuning(0, 0, 0, v),
                                  _assigned, lambda v: copy.copy(pm4g.BatchedTuning(launch=v, record_capacity=9))])
def test_a_named_launch_is_kept(hit, make, launch):
    got = _shape(make(launch))
    assert got[3] == launch
    if launch == 0 and hit is not None:
        assert got[:3] == (2048, 77, 99)


def test_no_named_launch(hit):
    want = (2048, 77, 99, hit["launch"]) if hit is not None else (0, 0, 0, 1)
    assert _shape(None) == want
    assert _shape(pm4g.BatchedTuning()) == want
    assert _shape(pm4g.BatchedTuning(pair_capacity=8, cell_capacity=3)) == want


def test_a_whole_shape_is_kept(hit):
    for launch in (0, 1):
        t = pm4g.BatchedTuning(tile_events=4096, emit_blocks=5, launch=launch, cell_capacity=11)
        assert _shape(t) == (4096, 5, 0, launch)
        assert pm4g._launch_shape(t, 20, 5, 1000).cell_capacity == 11
    assert _shape(pm4g.BatchedTuning(tile_events=4096)) == (4096, 0, 0, 0)


def test_the_callers_tuning_is_left_alone(hit):
    t = pm4g.BatchedTuning()
    pm4g._launch_shape(t, 20, 5, 1000)
    assert (t.tile_events, t.launch, t.launch_given) == (0, 0, False)
