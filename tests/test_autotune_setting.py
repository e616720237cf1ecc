"""The autotuner's candidates are timed under the setting that the batches run
under afterwards, and what is in force is one of them (no GPU: the timing
itself is replaced)."""
import json

import pytest
import torch

import paper_2204_03380_amd as rtm
from paper_2204_03380_amd import autotune

GRID2 = rtm.Grid(2, 10, 181, 1, 181, 10.0)
GRID3 = rtm.Grid(3, 10, 108, 108, 108, 10.0)


@pytest.fixture(autouse=True)
def _restore():
    snap = rtm.tuning_snapshot()
    yield
    rtm.tuning_restore(snap)
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 0, 0)


def _tune(monkeypatch, grid, seconds, **kw):
    calls = []

    def timed(fwd, rev, *rest):
        calls.append((fwd, rev, rtm.rtm_get_tuning(rtm.RTM_TUNE_EXACT)[0]))
        return seconds(len(calls) - 1)
    monkeypatch.setattr(autotune, "_time_shape", timed)
    res = autotune.tune_batch(grid, torch.zeros(1), torch.zeros(8), [None], [None], 1e-3, **kw)
    return res, calls


@pytest.mark.parametrize("grid", [GRID2, GRID3])
@pytest.mark.parametrize("exact", [0, 1])
def test_timed_under_the_setting_in_force(monkeypatch, grid, exact):
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, exact, 0)
    _, calls = _tune(monkeypatch, grid, lambda i: (1.0 + i, 1.0 + i))
    assert {c[2] for c in calls} == {exact}
    assert rtm.rtm_get_tuning(rtm.RTM_TUNE_EXACT)[0] == exact


@pytest.mark.parametrize("grid", [GRID2, GRID3])
def test_current_configuration_is_a_candidate_and_stays_unless_beaten(monkeypatch, grid):
    ops = (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM)
    before = [autotune.configured(op, grid.ndim) for op in ops]
    res, calls = _tune(monkeypatch, grid, lambda i: (2.0, 2.0))
    assert list(calls[0][:2]) == before and res["table"]["current"] == (2.0, 2.0)
    assert [autotune.configured(op, grid.ndim) for op in ops] == before
    res, calls = _tune(monkeypatch, grid, lambda i: (1.0 if i == 3 else 2.0, 1.0 if i == 4 else 2.0))
    assert autotune.configured(ops[0], grid.ndim) == calls[3][0] == res["forward"][:-1]
    assert autotune.configured(ops[1], grid.ndim) == calls[4][1] == res["reverse"][:-1]


@pytest.mark.parametrize("op", [rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM])
def test_library_defaults_are_among_the_3d_candidates(op):
    want = {rtm.RTM_OP_MODEL: (2, 16, 126), rtm.RTM_OP_RTM: (1, 8, 54)}[op]
    assert any(s[:3] == want for s in autotune.DEFAULT_SHAPES_3D)


def test_cached_choices_differ_by_setting(monkeypatch, tmp_path):
    path = str(tmp_path / "cache.json")
    timed = []
    for exact in (0, 1, 0, 1):
        rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, exact, 0)
        _, calls = _tune(monkeypatch, GRID2, lambda i: (1.0, 1.0), cache_path=path)
        timed.append(len(calls) > 0)
    assert timed == [True, True, False, False] and len(json.load(open(path))) == 2
