"""The filter's convolutions at the edges of their work split: one-channel
layers around blocks of four rows, the LDS-staged kernel around strips of 64
voxels, four rows and its z chunks."""
import numpy as np
import pytest
import torch

import oracle.unet as U
import paper_2204_03380_amd.unet as N

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bf(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(torch.bfloat16)


def _operands(shape, ci, co):
    rng = np.random.default_rng(ci + 100 * co)
    nv = int(np.prod(shape))
    x = U.bf16(rng.standard_normal((nv, ci)))
    w = rng.standard_normal((co, ci, 3, 3, 3)) * np.sqrt(2.0 / (27 * ci))
    skip = U.bf16(rng.standard_normal((nv, co)))
    wf = torch.empty((co, 27 * ci), dtype=torch.bfloat16, device=DEV)
    wb = torch.empty((ci, 27 * co), dtype=torch.bfloat16, device=DEV)
    wm = torch.from_numpy(np.ascontiguousarray(np.transpose(w.reshape(co, ci, 27), (0, 2, 1)), dtype=np.float32))
    N.weight_pack(wm.to(DEV), ci, co, wf, wb)
    return rng, x, U.bf16(w), rng.standard_normal(co).astype(np.float32), skip, wf, wb


def _conv(x, w, shape, b=None):
    """float64 convolution of channels-last x, and the sum of its terms' sizes."""
    n, d, h, s = shape
    t = torch.from_numpy(np.asarray(x, np.float64).reshape(n, d, h, s, -1)).permute(0, 4, 1, 2, 3)
    k = torch.from_numpy(np.ascontiguousarray(w, dtype=np.float64))
    f = lambda a, c: torch.nn.functional.conv3d(a, c, padding=1).permute(0, 2, 3, 4, 1).reshape(n * d * h * s, -1).numpy()
    y, size = f(t, k), f(t.abs(), k.abs())
    return (y, size) if b is None else (y + b, size + np.abs(b))


# float32 sums of 27 ci products (exact: bfloat16 factors) and the bias: at
# most 27 ci + 1 roundings of 2^-24 of the sum of sizes
def _check(y, ref, size, ci):
    assert np.all(np.abs(y.double().cpu().numpy() - ref) <= (27 * ci + 2) * 2.0 ** -24 * size)


@pytest.mark.parametrize("ci,co", [(1, 16), (16, 1)])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 1, 3, 5), (1, 2, 4, 64), (2, 3, 5, 67), (1, 2, 9, 1), (3, 4, 7, 33)])
def test_one_channel_layers(ci, co, shape):
    rng, x, w, b, skip, wf, wb = _operands(shape, ci, co)
    nv = x.shape[0]
    new = lambda c, t: torch.full((nv, c), 7.0, dtype=t, device=DEV)
    y, r, out = new(co, torch.float32), new(co, torch.bfloat16), new(co, torch.bfloat16)
    N.conv3d_fwd(shape, ci, co, _bf(x), wf, torch.from_numpy(b).to(DEV), False, skip=_bf(skip), y=y, r=r, out=out)
    _check(y, *_conv(x, w, shape, b), ci)
    assert torch.equal(r, y.to(torch.bfloat16)) and torch.equal(out, (y + _bf(skip).float()).to(torch.bfloat16))
    dy = U.bf16(rng.standard_normal((nv, co)))
    dx = new(ci, torch.float32)
    N.conv3d_dgrad(shape, ci, co, _bf(dy), wb, dx)
    _check(dx, *_conv(dy, np.flip(w, (2, 3, 4)).transpose(1, 0, 2, 3, 4), shape), co)


@pytest.mark.parametrize("ci,co", [(16, 32), (32, 16), (64, 32)])
@pytest.mark.parametrize("shape", [(8, 33, 5, 64), (5, 66, 1, 130), (3, 61, 8, 65)])
def test_lds_staged_edges(ci, co, shape):
    rng, x, w, b, skip, wf, wb = _operands(shape, ci, co)
    nv = x.shape[0]
    outs = []
    try:
        for lds in (True, False):
            N.set_conv_lds(lds)
            y = torch.full((nv, co), 7.0, device=DEV)
            r = torch.full((nv, co), 7.0, dtype=torch.bfloat16, device=DEV)
            out = torch.empty_like(r)
            N.conv3d_fwd(shape, ci, co, _bf(x), wf, torch.from_numpy(b).to(DEV), True, skip=_bf(skip), y=y, r=r, out=out)
            outs.append((y, r, out))
    finally:
        N.set_conv_lds(True)
    for p, q in zip(*outs):
        assert torch.equal(p, q)
    ref, size = _conv(x, w, shape, b)
    _check(outs[0][0], np.maximum(ref, 0.0), size, ci)


# Three samples together (3 x 2^18 voxels and more) take four rows per thread,
# each alone one row: the same bits, whatever is left of the last four rows.
@pytest.mark.parametrize("ci,co", [(1, 16), (16, 1)])
@pytest.mark.parametrize("d,h,w", [(56, 65, 73), (61, 66, 67), (58, 67, 71), (64, 64, 64)])
def test_one_channel_layers_rows_per_thread(ci, co, d, h, w):
    n, nv = 3, 3 * d * h * w
    assert nv // 3 < 3 << 18 <= nv
    rng, x, _, b, skip, wf, wb = _operands((n, d, h, w), ci, co)
    x, skip, dy, mask = _bf(x), _bf(skip), _bf(rng.standard_normal((nv, co))), _bf(rng.standard_normal((nv, ci)))
    bias = torch.from_numpy(b).to(DEV)

    def run(shape, at):
        k = int(np.prod(shape))
        y, r = torch.full((k, co), 7.0, device=DEV), torch.full((k, co), 7.0, dtype=torch.bfloat16, device=DEV)
        out, dx = torch.empty_like(r), torch.full((k, ci), 7.0, device=DEV)
        part = lambda a: a[at].clone()  # 16-byte aligned
        N.conv3d_fwd(shape, ci, co, part(x), wf, bias, True, skip=part(skip), y=y, r=r, out=out)
        N.conv3d_dgrad(shape, ci, co, part(dy), wb, dx)
        g = [torch.full((k, ci), 7.0, dtype=torch.bfloat16, device=DEV)] if ci == 16 else []
        for t in g:  # one channel has no fused ReLU gradient
            N.conv3d_dgrad(shape, ci, co, part(dy), wb, dx, mask=part(mask), g_out=t)
        return [y, r, out, dx] + g

    each = [run((1, d, h, w), slice(i * nv // n, (i + 1) * nv // n)) for i in range(n)]
    for k, t in enumerate(run((n, d, h, w), slice(0, nv))):
        assert torch.isfinite(t.float()).all() and torch.equal(t, torch.cat([e[k] for e in each])), k
