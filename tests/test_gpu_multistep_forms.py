"""Every form of the 2-D multi-step kernels against the one-step kernels, bit
for bit.  The form that a batch takes follows from its size; each test asks the
plan which one it got (BatchPlan.launch_shape), so that a changed rule cannot
leave a form untested unnoticed."""
import numpy as np
import pytest
import torch

import paper_2204_03380_amd as rtm
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OPS = {"model": rtm.RTM_OP_MODEL, "rtm": rtm.RTM_OP_RTM, "vjp": rtm.RTM_OP_VJP}
NT, NB = 7, 12


def _configure(exact, steps, vec, zseg):
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, int(exact), 0)
    for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM):
        rtm.rtm_set_tuning2d(op, vec, 1, zseg)
        rtm.rtm_set_steps_per_launch(op, steps)


class _Batch:
    """`shots` shots on one smooth model of NX x NZ padded cells, sources along
    the top, receivers in two lines (half cells: two and four nodes each)."""

    def __init__(self, NX, NZ):
        nx, nz = NX - 2 * NB, NZ - 2 * NB
        v = synth.random_model((nz, nx), 4, 1600, 3000, sigma=2.0)
        self.grid = rtm.Grid.for_model(v, 10.0, NB)
        self.vp = rtm.rtm_rbc_pad(self.grid, torch.from_numpy(v).to(DEV), 4, 0.0)
        self.w = torch.from_numpy(synth.ricker(25.0, 1e-3, NT, t0=0.3e-3 * NT)).to(DEV)
        xs = np.arange(0, nx - 1, 3) + 0.5
        self.rec = np.concatenate([synth.line_receivers(xs, 2.0), synth.line_receivers(xs, nz / 2 + 0.25)])
        g = torch.Generator(DEV).manual_seed(4)
        self.d = torch.randn((len(self.rec), NT + 1), generator=g, device=DEV)
        self.nx = nx

    def plan(self, op, shots):
        shape, key = {"model": ((len(self.rec), NT + 1), "traces_out"), "rtm": (self.grid.interior_shape, "image"),
                      "vjp": (self.grid.padded_shape, "grad_v_pad")}[op]
        outs = [torch.zeros(shape, device=DEV) for _ in range(shots)]
        items = []
        for i, o in enumerate(outs):
            src = np.array([(37.3 * (i + 1)) % (self.nx - 1), 0.0, 1.6], np.float32)
            items.append(rtm.BatchShot(self.grid, self.vp, self.w, src, self.rec, **{key: o},
                                       **({} if op == "model" else {"traces_in": self.d})))
        return rtm.BatchPlan(OPS[op], items, 1e-3, NT), outs

    def run(self, op, shots):
        plan, outs = self.plan(op, shots)
        shape = plan.launch_shape(op != "model")
        plan.run()
        torch.cuda.synchronize()
        plan.free()
        return outs, shape


def _compare(batch, op, shots, check):
    outs, shape = batch.run(op, shots)
    check(shape)
    _configure(True, 1, 2, 36)
    want, one = batch.run(op, shots)
    assert one["steps"] == 1
    assert any(o.any() for o in want)
    for a, b in zip(outs, want):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.fixture(scope="module")
def wide():
    return _Batch(1024, 512)


# Marching strips.  1024 x 512 cells: two shots take little of the memory-side
# cache, 8 at nine rows give 4096 tiles and more (rows loaded when they are due,
# not ahead), 33 exceed the cache (what is touched once goes past it).
@pytest.mark.parametrize("op", ["model", "rtm"])
@pytest.mark.parametrize("steps", [2, 3])
@pytest.mark.parametrize("vec", [1, 2, 4])
@pytest.mark.parametrize("shots,zseg", [(2, 9), (8, 9), (33, 9), (33, 108)])
def test_strips(wide, op, steps, vec, shots, zseg):
    _configure(True, steps, vec, zseg)
    own = 64 * vec - 8 * (steps - 1)
    tiles = shots * -(-1024 // own) * -(-513 // zseg)

    def check(s):
        assert (s["steps"], s["vec"], s["rows"], s["waves"], s["tiles"]) == (steps, vec, zseg, 0, tiles)
        assert s["uncached"] == (shots == 33 and vec < 4)
        if vec < 4:
            assert (tiles >= 4096) == (zseg == 9 and shots > 2)
    _compare(wide, op, shots, check)


# The gradient's strips: three steps where the runtime chooses, two as configured
@pytest.mark.parametrize("steps,vec,shots,uncached", [(3, 1, 8, 0), (3, 1, 33, 1), (3, 2, 12, 0), (3, 2, 33, 1), (3, 4, 24, 0),
                                                      (2, 1, 8, 0), (2, 1, 33, 1), (2, 2, 12, 0), (2, 2, 33, 1), (2, 4, 24, 0)])
def test_gradient_strips(wide, steps, vec, shots, uncached):
    _configure(False, steps, vec, 108)

    def check(s):
        assert (s["steps"], s["vec"], s["waves"], s["uncached"]) == (steps, vec, 0, uncached)
    _compare(wide, "vjp", shots, check)


@pytest.mark.parametrize("vec,shots,zseg", [(1, 2, 9), (2, 2, 9), (1, 33, 108), (2, 33, 108), (1, 8, 9), (2, 8, 9), (4, 2, 27)])
def test_gradient_strips_of_two_steps_ahead_and_not(wide, vec, shots, zseg):
    _configure(True, 2, vec, zseg)

    def check(s):
        assert (s["steps"], s["vec"], s["rows"], s["waves"]) == (2, vec, zseg, 0)
        if vec < 4:
            assert (s["tiles"] >= 4096) == (shots == 8)
    _compare(wide, "vjp", shots, check)


# models of 113 to 120 columns: one strip of two steps, not two of three
def test_narrow_gradient():
    batch = _Batch(117, 1891)
    _configure(False, 3, 2, 108)

    def check(s):
        assert (s["steps"], s["vec"], s["waves"]) == (2, 2, 0)
    _compare(batch, "vjp", 60, check)
# The block kernels: 8 wavefronts x 4 rows at one float per lane, 12 x 3 and
# 16 x 3 at two; one and several shots
@pytest.mark.parametrize("op", ["model", "rtm", "vjp"])
@pytest.mark.parametrize("steps,NX,NZ,shots,waves", [(2, 281, 281, 1, 8), (2, 281, 97, 3, 8), (2, 1400, 540, 1, 12),
                                                     (2, 700, 540, 2, 12), (2, 1574, 540, 1, 16), (3, 281, 281, 1, 8),
                                                     (3, 900, 540, 1, 12), (3, 880, 270, 2, 12), (3, 1574, 540, 1, 16)])
def test_blocks(op, steps, NX, NZ, shots, waves):
    batch = _Batch(NX, NZ)
    _configure(False, steps, 2, 108)

    def check(s):
        assert (s["steps"], s["waves"]) == (steps, waves)
    _compare(batch, op, shots, check)


# two reverse steps of a job with too many blocks of three
@pytest.mark.parametrize("op", ["rtm", "vjp"])
def test_blocks_of_two_steps_where_three_have_too_many(op):
    batch = _Batch(700, 380)
    _configure(False, 3, 2, 108)

    def check(s):
        assert (s["steps"], s["vec"], s["waves"]) == (2, 2, 16)
    _compare(batch, op, 8, check)
