"""3-D launches at the edges of tiles: whatever the shape, the tile order and
the treatment of arrays touched once, the results are the same bit for bit
(every cell takes the same operations)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2204_03380_amd as rtm
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES_F = [(v, ty, z) for v in (1, 2, 4) for ty in (4, 8, 16) for z in (9, 27) if v * ty < 64]
SHAPES_R = [(v, ty, z) for v, ty, z in SHAPES_F if ty < 16 or v == 1]


@pytest.fixture(autouse=True)
def _restore():
    ops = (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM)
    old = [rtm.rtm_get_tuning3d(op) for op in ops]
    yield
    for op, t in zip(ops, old):
        rtm.rtm_set_tuning3d(op, *t)
        rtm.rtm_set_tile_order3d(op, 0)
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 0, 0)


def _shot(nx, ny, nz, nb, nt, seed=3):
    v = synth.random_model((nz, ny, nx), seed, 1600, 3000, sigma=2.0)
    g = rtm.Grid.for_model(v, 10.0, nb)
    vp = rtm.rtm_rbc_pad(g, torch.from_numpy(v).to(DEV), seed, 0.0)
    top = np.array([nx - 1, ny - 1, nz - 1], np.float32)
    src = np.minimum(0.6 * top + 0.3, top).astype(np.float32)
    # receivers between grid points on a diagonal plane: every y tile and z band holds some
    n = 40
    rec = (np.linspace(0, 1, n)[:, None] * top[None]).astype(np.float32)
    w = torch.from_numpy(synth.ricker(25.0, 1e-3, nt, t0=0.3 * nt * 1e-3)).to(DEV)
    d = torch.randn((n, nt + 1), generator=torch.Generator(DEV).manual_seed(seed), device=DEV)
    return dict(grid=g, v_pad=vp, dt=1e-3, wavelet=w, src=src, rec=rec), d


def _all(shot, d):
    tr, p, q = rtm.rtm_model_shot(**shot, want_last=True)
    out = rtm.rtm_rtm_shot(**shot, traces=d, want_numden=True)
    st = rtm.rtm_storage_shot(shot["grid"], shot["v_pad"], shot["dt"], shot["wavelet"], shot["src"], shot["rec"], d, 3, 1,
                              want_numden=True)
    gv, gw = rtm.rtm_model_shot_vjp(**shot, grad_traces=d, want_wavelet_grad=True)
    return {"traces": tr, "p": p, "q": q, "num": out["num"], "den": out["den"], "snum": st["num"], "sden": st["den"],
            "snaps": st["snapshots"], "grad": gv, "grad_wavelet": gw}


def _same(a, b, what):
    for k in a:
        assert torch.isfinite(a[k]).all() and torch.equal(a[k], b[k]), (what, k)


@pytest.mark.parametrize("nx,ny,nz,nb,nt", [(1, 1, 1, 0, 4), (5, 3, 2, 4, 8), (56, 8, 10, 4, 12), (57, 9, 11, 4, 13),
                                            (121, 25, 20, 3, 11)])
def test_shapes_agree(nx, ny, nz, nb, nt):
    shot, d = _shot(nx, ny, nz, nb, nt)
    default = _all(shot, d)  # the shape a job chooses by itself
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 1, 0)
    rtm.rtm_set_tuning3d(rtm.RTM_OP_MODEL, 1, 4, 9)
    rtm.rtm_set_tuning3d(rtm.RTM_OP_RTM, 1, 4, 9)
    want = _all(shot, d)
    _same(default, want, "default")
    for i, f in enumerate(SHAPES_F):
        r = SHAPES_R[i % len(SHAPES_R)]
        rtm.rtm_set_tuning3d(rtm.RTM_OP_MODEL, *f)
        rtm.rtm_set_tuning3d(rtm.RTM_OP_RTM, *r)
        for op in (rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM):
            rtm.rtm_set_tile_order3d(op, i & 1)
        _same(_all(shot, d), want, (f, r))


# One shot of 200^3 padded cells keeps its arrays (96 MB forward, 206 reverse
# imaging, 192 gradient) in the memory-side cache, three together do not.
@pytest.mark.parametrize("op", [rtm.RTM_OP_MODEL, rtm.RTM_OP_RTM, rtm.RTM_OP_VJP])
def test_large_batch_equals_single(op):
    nt = 6
    shot, d = _shot(180, 180, 180, 10, nt)

    def run(n):
        g = shot["grid"]
        new = lambda shape: torch.zeros(shape, device=DEV)
        outs = [new((len(d), nt + 1) if op == rtm.RTM_OP_MODEL else
                    g.interior_shape if op == rtm.RTM_OP_RTM else g.padded_shape) for _ in range(n)]
        key = {rtm.RTM_OP_MODEL: "traces_out", rtm.RTM_OP_RTM: "image", rtm.RTM_OP_VJP: "grad_v_pad"}[op]
        shots = [rtm.BatchShot(g, shot["v_pad"], shot["wavelet"], shot["src"], shot["rec"],
                               traces_in=None if op == rtm.RTM_OP_MODEL else d, **{key: o}) for o in outs]
        plan = rtm.BatchPlan(op, shots, shot["dt"], nt)
        plan.run()
        torch.cuda.synchronize()
        plan.free()
        return outs

    one = run(1)[0]
    assert torch.isfinite(one).all() and one.any()
    for o in run(3):
        assert torch.equal(o, one)


@pytest.mark.timeout(300)
def test_storage_beyond_the_cache():
    """276^3 padded cells (252 MB a step): the forward and receiver passes
    against the oracle (its bound for this operation, rel-L2 1e-4; unit-scale
    wavelet, so that the short run is not dominated by near-zero values), and
    the receiver pass in small tiles."""
    nt, nb, seed, n = 6, 8, 3, 260
    v = synth.random_model((n, n, n), seed, 1600, 3000, sigma=2.0)
    g = rtm.Grid.for_model(v, 10.0, nb)
    vp = rtm.rtm_rbc_pad(g, torch.from_numpy(v).to(DEV), seed, 0.0)
    rng = np.random.default_rng(0)
    w = rng.standard_normal(nt).astype(np.float32)
    src = np.array([130.3, 129.6, 131.5], np.float32)
    rec = np.array([[128.5 + 4 * i, 130.0, 130.25] for i in range(-6, 7)], np.float32)
    d = rng.standard_normal((len(rec), nt + 1)).astype(np.float32)
    args = (g, vp, 1e-3, torch.from_numpy(w).to(DEV), src, rec, torch.from_numpy(d).to(DEV), 2, 1)
    x = rtm.rtm_storage_shot(*args, want_numden=True)
    vo = oracle.rbc_pad(v, nb, seed, 0.0)
    ref = oracle.rtm_storage_shot(vo, 10.0, nb, 1e-3, w.astype(np.float64), src, rec, d.astype(np.float64), 2, 1)
    rtm.rtm_set_tuning(rtm.RTM_TUNE_EXACT, 1, 0)
    rtm.rtm_set_tuning3d(rtm.RTM_OP_MODEL, 1, 4, 18)
    y = rtm.rtm_storage_shot(*args, want_numden=True)
    for k in ("num", "den"):
        assert torch.equal(x[k], y[k])
        a = x[k].cpu().numpy().astype(np.float64)
        assert a.any() and np.linalg.norm(a - ref[k]) < 1e-4 * np.linalg.norm(ref[k])
