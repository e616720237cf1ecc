"""2-D launches of two and three time steps: whatever the shape, the results
are those of the one-step kernels bit for bit (every cell takes the same
operations), modeling, imaging and gradient alike."""
import numpy as np
import pytest
import torch

import paper_2204_03380_amd as rtm
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _shot(nx, nz, nb, nt, rows=3, seed=3):
    """Smooth model, source between grid points near a corner, `rows` lines of
    receivers at half cells (several receiver nodes per column)."""
    v = synth.random_model((nz, nx), seed, 1600, 3000, sigma=2.0)
    g = rtm.Grid.for_model(v, 10.0, nb)
    vp = rtm.rtm_rbc_pad(g, torch.from_numpy(v).to(DEV), seed, 0.0)
    src = np.maximum(np.array([min(nx - 1.25, 0.6 * nx + 0.3), 0.0, min(nz - 1.5, 2.6)], np.float32), 0.0)
    zs = np.linspace(0.0, nz - 1.0, rows) if rows > 1 else [min(2.25, nz - 1.0)]
    xs = np.minimum(np.arange(nx) + 0.5, nx - 1.0)
    rec = np.concatenate([synth.line_receivers(xs, float(z)) for z in zs])
    w = torch.from_numpy(synth.ricker(25.0, 1e-3, nt, t0=0.3 * nt * 1e-3)).to(DEV)
    d = torch.randn((len(rec), nt + 1), generator=torch.Generator(DEV).manual_seed(seed), device=DEV)
    return dict(grid=g, v_pad=vp, dt=1e-3, wavelet=w, src=src, rec=rec), d


def _all(shot, d):
    tr, p, q = rtm.rtm_model_shot(**shot, want_last=True)
    out = rtm.rtm_rtm_shot(**shot, traces=d, want_numden=True)
    gv, gw = rtm.rtm_model_shot_vjp(**shot, grad_traces=d, want_wavelet_grad=True)
    return {"traces": tr, "p_last": p, "p_prev": q, "image": out["image"], "num": out["num"], "den": out["den"], "grad": gv,
            "grad_wavelet": gw}


def _shape(exact, steps, vec=2, zseg=108):
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, int(exact), 0)
    for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM):
        rtm.rtm_set_tuning2d(op, vec, 1, zseg)
        rtm.rtm_set_steps_per_launch(op, steps)


def _same(a, b):
    for k in a:
        assert torch.isfinite(a[k]).all() and torch.equal(a[k], b[k]), k


# grids around the edges of strips (48 .. 248 owned columns) and of nine-row
# tiles, more receivers in a tile than a wavefront holds at once, and step
# counts that leave one and two steps over
@pytest.mark.parametrize("nx,nz,nb,nt", [(1, 1, 0, 4), (9, 7, 4, 7), (104, 46, 4, 8), (105, 45, 4, 9), (233, 91, 7, 11),
                                         (300, 130, 9, 20)])
def test_configured_shapes(nx, nz, nb, nt):
    shot, d = _shot(nx, nz, nb, nt)
    _shape(True, 1)
    want = _all(shot, d)
    for steps in (2, 3):
        for vec, zseg in ((1, 9), (1, 27), (2, 9), (2, 54), (4, 18)):
            _shape(True, steps, vec, zseg)
            _same(want, _all(shot, d))


# shapes the runtime chooses: one strip, few and many tiles
@pytest.mark.parametrize("nx,nz,nb,nt", [(33, 21, 5, 10), (201, 201, 40, 31), (420, 330, 30, 10), (1574, 534, 0, 7),
                                         (2301, 751, 60, 8)])
def test_chosen_shapes(nx, nz, nb, nt):
    shot, d = _shot(nx, nz, nb, nt, rows=1)
    _shape(True, 1)
    want = _all(shot, d)
    for steps in (2, 3):
        _shape(False, steps)
        _same(want, _all(shot, d))


# enough tiles for the kernels that load each row when it is due (from 4096
# tiles on), and, just below, for those that load it three rows ahead
@pytest.mark.parametrize("shots", [48, 49])
@pytest.mark.parametrize("steps", [2, 3])
def test_many_tiles(shots, steps):
    shot, d = _shot(301, 101, 10, 7, rows=1)
    own = 64 - 8 * (steps - 1)
    assert (shots * -(-321 // own) * 14 >= 4096) == (shots == 49 or steps == 3)
    g = shot["grid"]

    def run():
        def desc(i, **kw):
            src = np.array([20.0 + 5 * i, 0.0, 2.0], np.float32)
            return rtm.BatchShot(g, shot["v_pad"], shot["wavelet"], src, shot["rec"], **kw)
        tr = torch.zeros((shots,) + tuple(d.shape), device=DEV)
        im = torch.zeros((shots,) + tuple(g.interior_shape), device=DEV)
        gv = torch.zeros((shots,) + tuple(g.padded_shape), device=DEV)
        for op, kw in ((rtm.RTM_OP_MODEL, lambda i: dict(traces_out=tr[i])), (rtm.RTM_OP_RTM, lambda i: dict(traces_in=d, image=im[i])),
                       (rtm.RTM_OP_VJP, lambda i: dict(traces_in=d, grad_v_pad=gv[i]))):
            rtm.BatchPlan(op, [desc(i, **kw(i)) for i in range(shots)], 1e-3, 7).run()
        return {"traces": tr, "image": im, "grad": gv}
    _shape(True, 1)
    want = run()
    _shape(True, steps, 1, 9)
    _same(want, run())


# the block kernels' three shapes (small jobs): edges of the 48 x 16, 112 x 20
# and 112 x 32 cells a block of three steps owns (56 x 24, 120 x 28 and
# 120 x 40 with two), more receiver nodes in a block than it has threads, all
# wavefronts of the last block idle but one
@pytest.mark.parametrize("nx,nz,nb,nt,rows", [(1, 1, 0, 3, 1), (48, 16, 0, 6, 3), (49, 17, 0, 7, 3), (57, 47, 4, 8, 24),
                                              (800, 450, 40, 7, 2), (785, 460, 0, 9, 1), (1121, 512, 0, 6, 1),
                                              (1100, 513, 10, 8, 3), (2000, 600, 50, 7, 1)])
def test_block_kernels(nx, nz, nb, nt, rows):
    shot, d = _shot(nx, nz, nb, nt, rows=rows)
    _shape(True, 1)
    want = _all(shot, d)
    for steps in (2, 3):
        _shape(False, steps)
        _same(want, _all(shot, d))


def test_block_kernels_uneven_batch():
    """Blocks of several shots of different grids in one launch."""
    shots = [_shot(nx, nz, 5, 8, rows=2, seed=i) for i, (nx, nz) in enumerate([(90, 61), (201, 30), (33, 140)])]

    def run():
        tr = [torch.zeros_like(d) for _, d in shots]
        im = [torch.zeros(s["grid"].interior_shape, device=DEV) for s, _ in shots]
        gv = [torch.zeros(s["grid"].padded_shape, device=DEV) for s, _ in shots]
        keys = ("grid", "v_pad", "wavelet", "src", "rec")
        for op, kw in ((rtm.RTM_OP_MODEL, lambda i: dict(traces_out=tr[i])),
                       (rtm.RTM_OP_RTM, lambda i: dict(traces_in=shots[i][1], image=im[i])),
                       (rtm.RTM_OP_VJP, lambda i: dict(traces_in=shots[i][1], grad_v_pad=gv[i]))):
            rtm.BatchPlan(op, [rtm.BatchShot(*(s[k] for k in keys), **kw(i)) for i, (s, _) in enumerate(shots)], 1e-3, 8).run()
        return {f"{n}{i}": t for n, ts in (("traces", tr), ("image", im), ("grad", gv)) for i, t in enumerate(ts)}
    _shape(True, 1)
    want = run()
    _shape(False, 3)
    _same(want, run())


# Ten shots of 2401 x 851 padded cells exceed the memory-side cache (335 MB
# forward, 790 reverse), one does not: the kernels that keep what they touch
# once out of the caches give the bits of the others.
@pytest.mark.parametrize("op", [rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM, rtm.RTM_OP_VJP])
@pytest.mark.parametrize("steps", [2, 3])
def test_large_batch_equals_single(op, steps):
    nt = 7
    shot, d = _shot(2301, 751, 50, nt, rows=1)
    _shape(False, steps)

    def run(n):
        g = shot["grid"]
        shape = {rtm.RTM_OP_MODEL: (len(d), nt + 1), rtm.RTM_OP_RTM: g.interior_shape, rtm.RTM_OP_VJP: g.padded_shape}[op]
        key = {rtm.RTM_OP_MODEL: "traces_out", rtm.RTM_OP_RTM: "image", rtm.RTM_OP_VJP: "grad_v_pad"}[op]
        outs = [torch.zeros(shape, device=DEV) for _ in range(n)]
        plan = rtm.BatchPlan(op, [rtm.BatchShot(g, shot["v_pad"], shot["wavelet"], shot["src"], shot["rec"],
                                                traces_in=None if op == rtm.RTM_OP_MODEL else d, **{key: o})
                                  for o in outs], shot["dt"], nt)
        plan.run()
        torch.cuda.synchronize()
        plan.free()
        return outs

    try:
        one, many = run(1)[0], run(10)
    finally:
        _shape(False, 3)
    assert torch.isfinite(one).all() and one.any()
    for o in many:
        assert torch.equal(o, one)
