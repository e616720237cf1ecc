"""What a plan's passes launch (rtm_batch_shape): planning is host work, so
the choice of launch shapes is checked without a GPU; device addresses are
never dereferenced."""
import ctypes

import numpy as np
import pytest

import paper_2204_03380_amd as rtm
from paper_2204_03380_amd import _lib


@pytest.fixture(autouse=True)
def _defaults():
    snap = rtm.tuning_snapshot()
    for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM):
        rtm.rtm_set_tuning2d(op, 2, 1, 108)
        rtm.rtm_set_steps_per_launch(op, 3)
    rtm.rtm_set_tuning3d(rtm.RTM_OP_MODEL, 2, 16, 126)
    rtm.rtm_set_tuning3d(rtm.RTM_OP_RTM, 1, 8, 54)
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 0, 0)
    yield
    rtm.tuning_restore(snap)


def shape_of(op, padded, shots=1, reverse=False, shared=True, flags=0):
    """Shape of a batch of `shots` shots, padded extents (z, x) or (z, y, x)."""
    lib = _lib.load()
    nz, ny, nx = padded if len(padded) == 3 else (padded[0], 1, padded[1])
    grid = rtm.Grid(len(padded), nx, ny, nz, 10.0, 0)
    rec = np.zeros((1, 3), np.float32)
    descs = (_lib.RtmShotDesc * shots)()
    for i, d in enumerate(descs):
        d.grid = grid.c()
        d.v_pad = 0x10000 + (0 if shared else 0x10000 * i)
        d.wavelet = d.traces_in = d.traces_out = d.image = d.grad_v_pad = 0x10000
        d.nrec, d.rec = 1, rec.ctypes.data
    plan, ws = ctypes.c_void_p(), ctypes.c_size_t()
    _lib.check(lib.rtm_batch_plan(op, shots, descs, 1e-3, 20, 1e-3, flags, ctypes.byref(plan), ctypes.byref(ws)))
    s = _lib.RtmLaunchShape()
    try:
        _lib.check(lib.rtm_batch_shape(plan, int(reverse), ctypes.byref(s)))
    finally:
        lib.rtm_batch_free(plan)
    return {n: int(getattr(s, n)) for n, _ in s._fields_}


def test_query_reports_what_runs_not_what_is_configured():
    # two shots of 2421 x 871 take two reverse steps at one float, not the configured three at two
    assert rtm.rtm_get_steps_per_launch(rtm.RTM_OP_RTM) == 3 and rtm.rtm_get_tuning2d(rtm.RTM_OP_RTM)[0] == 2
    s = shape_of(rtm.RTM_OP_RTM, (871, 2421), 2, reverse=True)
    assert (s["steps"], s["vec"], s["waves"]) == (2, 1, 0)
    # a small job takes block kernels, a survey marching strips past the caches
    assert shape_of(rtm.RTM_OP_MODEL, (281, 281))["waves"] == 8
    s = shape_of(rtm.RTM_OP_MODEL, (871, 2421), 48)
    assert (s["steps"], s["vec"], s["rows"], s["waves"], s["uncached"]) == (3, 2, 108, 0, 1)
    # under RTM_TUNE_EXACT the configured shape runs
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 1, 0)
    rtm.rtm_set_tuning2d(rtm.RTM_OP_MODEL, 1, 1, 36)
    s = shape_of(rtm.RTM_OP_MODEL, (281, 281))
    assert (s["steps"], s["vec"], s["rows"], s["waves"], s["tiles"]) == (3, 1, 36, 0, 6 * 8)
    rtm.rtm_set_steps_per_launch(rtm.RTM_OP_MODEL, 1)
    rtm.rtm_set_tuning2d(rtm.RTM_OP_MODEL, 1, 4, 36)
    s = shape_of(rtm.RTM_OP_MODEL, (281, 281))
    assert (s["steps"], s["tx"], s["tiles"]) == (1, 4, 2 * 8)
    # persistent passes step once per item
    assert shape_of(rtm.RTM_OP_MODEL, (281, 281), flags=rtm.RTM_F_PERSISTENT)["steps"] == 1


def test_query_validation():
    lib = _lib.load()
    s = _lib.RtmLaunchShape()
    assert lib.rtm_batch_shape(None, 0, ctypes.byref(s)) == _lib.RTM_EINVAL
    with pytest.raises(rtm.RtmError):
        shape_of(rtm.RTM_OP_MODEL, (50, 50), reverse=True)
    with pytest.raises(rtm.RtmError):
        shape_of(rtm.RTM_OP_RTM, (50, 50), reverse=2)


# Sizes are padded (z, y, x).  Tiles of 16 rows (64 columns: a chip a quarter
# full) made the forward step of 64^3 cells 14.1 us instead of 7.1, and the
# receiver step of 144^3 18.1 instead of 12.0.
@pytest.mark.parametrize("padded,shots", [((64, 64, 64), 1), ((216, 46, 46), 1), ((46, 46, 216), 1), ((144, 144, 144), 1),
                                          ((188, 188, 188), 2), ((156, 156, 156), 3), ((124, 124, 124), 8),
                                          ((64, 64, 64), 16), ((9, 5, 3), 1)])
def test_forward_steps_in_the_cache_take_the_smallest_tiles(padded, shots):
    s = shape_of(rtm.RTM_OP_MODEL, padded, shots)
    assert (s["vec"], s["ty"], s["rows"], s["uncached"]) == (1, 4, 9, 0)


@pytest.mark.parametrize("padded,shots,tile", [((64, 64, 64), 1, (4, 9)), ((70, 90, 400), 1, (4, 9)), ((64, 64, 64), 16, (4, 18)),
                                               ((100, 180, 260), 1, (4, 27)), ((24, 353, 78), 3, (8, 9)), ((188, 188, 188), 1, (4, 27)),
                                               ((200, 200, 200), 1, (8, 18)), ((156, 156, 156), 4, (8, 9))])
@pytest.mark.parametrize("op", [rtm.RTM_OP_RTM, rtm.RTM_OP_VJP])
def test_reverse_steps_in_the_cache_keep_their_workgroups_resident(op, padded, shots, tile):
    s = shape_of(op, padded, shots, reverse=True)
    if not s["uncached"]:
        assert (s["vec"], s["ty"], s["rows"]) == (1, *tile)
        assert tile[0] == 8 or s["tiles"] <= 256 * (5.1 if tile[1] == 9 else 4.15)


@pytest.mark.parametrize("op,reverse,padded,shots,shared,uncached", [
    # one large grid: its model is touched once
    (rtm.RTM_OP_MODEL, False, (356, 612, 612), 1, True, 1), (rtm.RTM_OP_RTM, True, (356, 612, 612), 1, True, 1),
    (rtm.RTM_OP_VJP, True, (356, 612, 612), 1, True, 1), (rtm.RTM_OP_RTM, True, (252, 252, 252), 2, True, 1),
    # shots that share a model read it several times
    (rtm.RTM_OP_MODEL, False, (188, 188, 188), 8, True, 0), (rtm.RTM_OP_MODEL, False, (188, 188, 188), 8, False, 1),
    (rtm.RTM_OP_VJP, True, (188, 188, 188), 8, True, 0), (rtm.RTM_OP_VJP, True, (188, 188, 188), 8, False, 1),
    (rtm.RTM_OP_VJP, True, (96, 96, 96), 16, True, 1),
    (rtm.RTM_OP_RTM, True, (43, 337, 304), 4, True, 1),
    (rtm.RTM_OP_RTM, True, (124, 124, 124), 16, True, 0), (rtm.RTM_OP_RTM, True, (124, 124, 124), 16, False, 1),
    (rtm.RTM_OP_RTM, True, (188, 188, 188), 8, True, 0), (rtm.RTM_OP_RTM, True, (188, 188, 188), 8, False, 1)])
def test_arrays_kept_out_of_the_cache(op, reverse, padded, shots, shared, uncached):
    assert shape_of(op, padded, shots, reverse, shared)["uncached"] == uncached


# Three steps of a strip own 112 columns, two 120: models of 113 to 120 columns
# would march everything twice (60 shots of 117 x 1891: 118.5 us per step
# against 95.5, the older kernels 104.5).
@pytest.mark.parametrize("nx,steps", [(112, 3), (113, 2), (120, 2), (121, 3), (240, 3)])
def test_gradient_steps_of_narrow_models(nx, steps):
    assert shape_of(rtm.RTM_OP_VJP, (1891, nx), 60, reverse=True, shared=False)["steps"] == steps


def test_two_reverse_steps_take_blocks_before_nine_row_strips():
    for op in (rtm.RTM_OP_RTM, rtm.RTM_OP_VJP):
        s = shape_of(op, (1891, 112), 10, reverse=True)
        assert (s["steps"], s["vec"], s["rows"], s["waves"]) == (2, 2, 40, 16)


# The marches take nine rows (planes) a round without a check of each; only
# the block kernels' tiles, which hold all their rows at once, have any number.
@pytest.mark.parametrize("padded", [(9, 5), (201, 201), (434, 1474), (500, 880), (871, 2421), (1891, 117), (64, 64, 64),
                                    (156, 156, 156), (356, 612, 612)])
@pytest.mark.parametrize("shots", [1, 3, 12, 48])
@pytest.mark.parametrize("steps", [1, 2, 3])
def test_marching_tiles_are_whole_rounds(padded, shots, steps):
    for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM):
        rtm.rtm_set_steps_per_launch(op, steps)
    for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM, rtm.RTM_OP_VJP):
        for reverse in (False, True)[:1 + (op != rtm.RTM_OP_MODEL)]:
            s = shape_of(op, padded, shots, reverse)
            if s["waves"] == 0 or len(padded) == 3:
                assert s["rows"] > 0 and s["rows"] % 9 == 0
            else:
                rows = {8: 4, 12: 3, 16: 3}[s["waves"]]
                assert s["steps"] > 1 and s["rows"] == s["waves"] * rows - 8 * (s["steps"] - 1)


# us per step: 50 own models of 76 x 324 x 54 imaging 1046 -> 794 (older kernels
# 850), 30 shots on one model of 92 x 107 x 56 230 -> 186 (210)
@pytest.mark.parametrize("nx,shared,op,uncached", [
    (64, False, rtm.RTM_OP_RTM, 0), (65, False, rtm.RTM_OP_RTM, 1), (64, True, rtm.RTM_OP_RTM, 0),
    (64, True, rtm.RTM_OP_VJP, 0), (64, False, rtm.RTM_OP_VJP, 1), (40, False, rtm.RTM_OP_RTM, 0)])
def test_reverse_steps_of_one_strip_keep_to_the_caches(nx, shared, op, uncached):
    s = shape_of(op, (76, 324, nx), 10 if shared else 50, reverse=True, shared=shared)
    assert (s["uncached"], s["rows"]) == (uncached, 9)


@pytest.mark.parametrize("op,reverse,padded,shots,rows", [
    (rtm.RTM_OP_RTM, True, (195, 135, 125), 14, 9), (rtm.RTM_OP_VJP, True, (195, 135, 125), 14, 9),
    (rtm.RTM_OP_RTM, True, (200, 380, 380), 1, 9), (rtm.RTM_OP_RTM, True, (235, 501, 501), 1, 27),
    (rtm.RTM_OP_RTM, True, (356, 612, 612), 1, 54), (rtm.RTM_OP_MODEL, False, (356, 612, 612), 1, 72),
    (rtm.RTM_OP_MODEL, False, (390, 35, 50), 50, 9), (rtm.RTM_OP_MODEL, False, (76, 324, 54), 50, 9)])
def test_planes_per_tile_of_many_workgroups(op, reverse, padded, shots, rows):
    assert shape_of(op, padded, shots, reverse, shared=False)["rows"] == rows


@pytest.mark.parametrize("ny,ty", [(35, 4), (36, 4), (37, 8), (40, 8), (44, 8), (4, 4), (9, 4)])
def test_rows_of_reverse_tiles_on_few_rows(ny, ty):
    for op in (rtm.RTM_OP_RTM, rtm.RTM_OP_VJP):
        s = shape_of(op, (390, ny, 200), 50, reverse=True, shared=False)
        assert (s["ty"], s["rows"]) == (ty, 9)
