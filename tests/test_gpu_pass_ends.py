"""What a pass does once, before and after its time loop: velocity range,
trace transposes, zeroed fields, image finalisation over a batch, padding
adjoint."""
import numpy as np
import pytest
import torch

import oracle
import paper_2204_03380_amd as rtm
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one cell, lines, more columns than a wavefront, a corner of many terms
# (2-D: 41^2; 3-D: 13^3) and an edge of some (13^2)
@pytest.mark.parametrize("shape,nb,taper,fs", [((1, 1), 3, 0.0, False), ((1, 70), 9, 0.0, False), ((3, 2), 40, 0.0, False),
                                               ((67, 130), 40, 0.0, False), ((9, 300), 12, 0.5, True),
                                               ((1, 1, 1), 4, 0.0, False), ((2, 3, 70), 12, 0.5, False),
                                               ((9, 8, 7), 12, 0.0, True)])
def test_pad_adjoint_cells(shape, nb, taper, fs):
    rng = np.random.default_rng(5)
    v = rng.uniform(1500, 3000, shape).astype(np.float32)
    g = rtm.Grid.for_model(v, 10.0, nb)
    gp = rng.standard_normal(g.padded_shape).astype(np.float32)
    t = lambda a: torch.from_numpy(a).to(DEV)
    got = rtm.rtm_pad_adjoint(g, t(v), 31, 2600.0, t(gp), free_surface=fs, taper=taper).cpu().numpy()
    ref = oracle.pad_adjoint(v, nb, 31, 2600.0, gp.astype(np.float64), free_surface=fs, taper=taper)
    # m terms of float32, each rounded a few times: (m + 4) 2^-24 of the sum of their sizes
    size = oracle.pad_adjoint(v, nb, 31, 2600.0, np.abs(gp).astype(np.float64), free_surface=fs, taper=taper)
    m = (2 * nb + 1) ** len(shape)
    assert np.all(np.abs(got - ref) <= (m + 4) * 2.0 ** -24 * size)


@pytest.mark.parametrize("shape", [(1, 1), (7, 33), (131, 517), (40, 37, 30)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -1.0])
def test_velocity_range_sees_every_cell(shape, bad):
    g = rtm.Grid.for_model(np.zeros(shape, np.float32), 10.0, 0)
    w = torch.zeros(2, device=DEV)
    rec = np.zeros((1, 3), np.float32)
    n = int(np.prod(shape))
    for at in sorted({0, n // 2, n - 1}):
        v = torch.full((n,), 2000.0, device=DEV)
        v[at] = bad
        with pytest.raises(rtm.RtmError):
            rtm.rtm_model_shot(g, v.reshape(g.padded_shape), 1e-3, w, np.zeros(3, np.float32), rec)
    v = torch.full((n,), 2000.0, device=DEV)
    rtm.rtm_model_shot(g, v.reshape(g.padded_shape), 1e-3, w, np.zeros(3, np.float32), rec)


def _shots(ndim):
    """Four shots on two grids, each with its own number of receivers."""
    out = []
    for i, n in enumerate((70, 70, 45, 70)):
        shape = (31, n) if ndim == 2 else (20, 11, n)
        v = synth.random_model(shape, 3 + (n == 45), 1600, 3000, sigma=2.0)
        g = rtm.Grid.for_model(v, 10.0, 5)
        vp = rtm.rtm_rbc_pad(g, torch.from_numpy(v).to(DEV), 3, 0.0)
        nrec = (33, 1, 64, 20)[i]
        rec = np.stack([np.linspace(0, n - 1, nrec), np.zeros(nrec) + (3.5 if ndim == 3 else 0.0), np.zeros(nrec) + 1.5], 1)
        src = np.array([5.3 + 9 * i, 4.0 if ndim == 3 else 0.0, 7.7], np.float32)
        out.append((g, vp, src, rec.astype(np.float32), nrec))
    return out


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("accumulate", [True, False])
def test_batch_finalisation(ndim, accumulate):
    nt = 37
    w = torch.from_numpy(synth.ricker(25.0, 1e-3, nt, t0=0.01)).to(DEV)
    gen = torch.Generator(DEV).manual_seed(1)
    shots = _shots(ndim)
    data = [torch.randn((s[4], nt + 1), generator=gen, device=DEV) for s in shots]
    flags = rtm.RTM_F_ACCUMULATE if accumulate else 0

    def plan(op, items, flags=0):
        p = rtm.BatchPlan(op, items, 1e-3, nt, flags=flags)
        p.run()
        torch.cuda.synchronize()
        p.free()

    # modeling: the batch's traces are each shot's own
    both = [torch.full((s[4], nt + 1), 7.0, device=DEV) for s in shots]
    plan(rtm.RTM_OP_MODEL, [rtm.BatchShot(*s[:2], w, *s[2:4], traces_out=t) for s, t in zip(shots, both)])
    for s, t in zip(shots, both):
        assert torch.equal(t, rtm.rtm_model_shot(s[0], s[1], 1e-3, w, s[2], s[3]))
    # imaging: shots 0, 1 and 3 share an image, shot 2 stands between them
    def start():
        return [torch.full(shots[i][0].interior_shape, 0.25, device=DEV) for i in (0, 2)]
    which = (0, 0, 1, 0)
    got, want = start(), start()
    plan(rtm.RTM_OP_RTM, [rtm.BatchShot(*s[:2], w, *s[2:4], traces_in=d, image=got[k])
                          for s, d, k in zip(shots, data, which)], flags)
    for s, d, k in zip(shots, data, which):
        plan(rtm.RTM_OP_RTM, [rtm.BatchShot(*s[:2], w, *s[2:4], traces_in=d, image=want[k])], flags)
    for a, b in zip(got, want):
        assert torch.isfinite(a).all() and a.any() and torch.equal(a, b)
