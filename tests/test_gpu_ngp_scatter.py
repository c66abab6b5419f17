"""Neural-texture backward at the edges of its table scatter: windows of one and of several 16-vertex tiles, the largest
window and the ones past it, textures next to a tile's size, one to sixteen levels; and a gradient that is not finite,
which reaches the parameters of its own texel's vertices only."""
import numpy as np
import pytest

import scenes as S
from oracle import ngp as N
from vs_testlib import GRAD_RTOL, say

pytestmark = pytest.mark.gpu


def _run(res, log2, sizes, gt):
    import torch
    import paper_2409_02482_amd as P
    assert torch.cuda.is_available()
    cfg = P.NgpConfig(res, log2)
    params = [S.ngp_params(57 + l, l, len(res), log2) for l in range(len(sizes))]
    dev = [torch.from_numpy(p).cuda() for p in params]
    ws = P.ngp_workspace(cfg, sizes)
    tex = P.ngp_bake(dev, cfg, sizes, ws=ws)
    grads = P.ngp_backward(dev, cfg, sizes, tex, [torch.from_numpy(g).cuda() for g in gt], ws)
    torch.cuda.synchronize()
    return params, [g.cpu().numpy().astype(np.float64) for g in grads]


@pytest.mark.parametrize("res,log2,sizes", [
    ([1], 6, [(1, 1), (16, 16)]),
    ([2, 15, 16, 17], 10, [(16, 16), (17, 16), (15, 33)]),
    # 16 texels span 23, 24 and 25 vertices; twice and three times as many vertices as texels
    ([33, 44, 46, 48, 64, 96], 9, [(32, 32), (32, 80), (90, 32)]),
    (list(range(3, 67, 4)), 8, [(50, 31)]),
])
def test_scatter_windows(res, log2, sizes):
    rng = np.random.default_rng(41)
    gt = [rng.uniform(-1, 1, (h, w, 4)).astype(np.float32) for w, h in sizes]
    say(f"[gpu] ngp scatter res {res} sizes {sizes}")
    params, grads = _run(res, log2, sizes, gt)
    ocfg = N.NgpConfig(res, log2)
    for l, (w, h) in enumerate(sizes):
        want = N.backward(params[l].astype(np.float64), ocfg, w, h, gt[l].astype(np.float64))
        for name in ("tables", "W1", "b1", "W2", "b2", "W3", "b3"):
            o, s = N.param_layout(ocfg)[name]
            a, b = grads[l][o:o + int(np.prod(s))], want[o:o + int(np.prod(s))]
            assert np.abs(a - b).max() <= GRAD_RTOL * max(np.abs(b).max(), 1e-30), (l, name)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_gradient_that_is_not_finite_stays_with_its_texel(bad):
    res, log2, (w, h), (i, j) = [3, 9, 21, 40], 12, (40, 24), (19, 17)
    rng = np.random.default_rng(42)
    gt = rng.uniform(-1, 1, (h, w, 4)).astype(np.float32)
    gt[j, i] = 0.0
    _, clean = _run(res, log2, [(w, h)], [gt])
    gt[j, i, 1] = bad
    say(f"[gpu] ngp scatter with {bad}")
    _, got = _run(res, log2, [(w, h)], [gt])
    T, hit = 1 << log2, np.zeros((len(res), 1 << log2), bool)
    for lv, n in enumerate(res):
        x, y = int(np.floor((i + 0.5) / w * n)), int(np.floor((j + 0.5) / h * n))
        for dx in (0, 1):
            for dy in (0, 1):
                hit[lv, N.vertex_index(np.array([x + dx]), np.array([y + dy]), n, T)] = True
    hit = np.repeat(hit.reshape(-1), 2)
    tables = got[0][:hit.size]
    assert not np.isfinite(tables[hit]).any()
    assert np.abs(tables[~hit] - clean[0][:hit.size][~hit]).max() <= GRAD_RTOL * np.abs(clean[0][:hit.size]).max()


def test_gradients_whose_sums_overflow_stay_with_their_vertices():
    """Finite gradients near the largest float: a vertex whose sum fits a float has it, entries that no texel reaches stay
    zero, next to coarse levels where a tile's column alone overflows.  The texture ends inside its last tiles."""
    import torch
    import paper_2409_02482_amd as P
    res, log2, (w, h) = [1, 3, 9, 40, 60], 12, (40, 24)
    ocfg = N.NgpConfig(res, log2)
    params = S.ngp_params(57, 0, len(res), log2)
    o1, s1 = N.param_layout(ocfg)["W1"]
    params[:o1] *= np.float32(2.0 ** -4)      # the same network from smaller features: dL/de is 16 times as large
    params[o1:o1 + int(np.prod(s1))] *= np.float32(2.0 ** 4)
    f, Q = N.forward(params, ocfg, *N.texel_centres(w, h)), N.unpack(params, ocfg)
    gt = np.random.default_rng(43).uniform(0.5, 1, (h, w, 4)).astype(np.float32)

    def de_of(g):
        d0 = g.reshape(-1, 4).astype(np.float64) * f["t"] * (1.0 - f["t"])
        return ((((d0 @ Q["W3"]) * (f["z2"] > 0)) @ Q["W2"]) * (f["z1"] > 0)) @ Q["W1"]

    gt *= np.float32(2.5e38 / np.abs(de_of(gt)).max())
    de = de_of(gt)
    want, total = np.zeros((len(res), 1 << log2, 2)), np.zeros((len(res), 1 << log2, 2))
    for lv, (idx, wts) in enumerate(f["corners"]):
        for q, wt in zip(idx, wts):
            for c in range(2):
                np.add.at(want[lv, :, c], q, wt * de[:, 2 * lv + c])
                np.add.at(total[lv, :, c], q, np.abs(wt * de[:, 2 * lv + c]))
    fx = (np.arange(16) + 0.5) / w   # level 0: one cell, the first tile's columns into its left vertices
    assert np.abs(((1 - fx)[:, None] * de.reshape(h, w, -1)[:, :16, :2]).sum(1)).max() > 3.5e38
    fits = total < 3e38
    assert (np.abs(want) > 3.5e38).any() and (fits & (total > 0)).sum() > 1000   # both kinds are there
    cfg = P.NgpConfig(res, log2)
    say("[gpu] ngp scatter with sums that overflow")
    dev, ws = [torch.from_numpy(params).cuda()], P.ngp_workspace(cfg, [(w, h)])
    tex = P.ngp_bake(dev, cfg, [(w, h)], ws=ws)
    got = P.ngp_backward(dev, cfg, [(w, h)], tex, [torch.from_numpy(gt).cuda()], ws)[0].cpu().numpy().astype(np.float64)
    got = got[:want.size].reshape(want.shape)
    assert np.isfinite(got[fits]).all()
    assert np.abs(got - want)[fits].max() <= GRAD_RTOL * total[fits].max()
    assert (got[total == 0] == 0).all()


def test_texels_outside_the_texture_have_no_gradient():
    """A unit that is off at every texel but on for an all-zero encoding, with an infinite weight behind it: the texels that
    fill a tile up must not bring it into the gradients."""
    import torch
    import paper_2409_02482_amd as P
    res, log2, (w, h) = [3, 9], 8, (19, 18)
    ocfg, cfg = N.NgpConfig(res, log2), P.NgpConfig(res, log2)
    lay = N.param_layout(ocfg)
    params = S.ngp_params(57, 0, len(res), log2)

    def part(name):
        o, s = lay[name]
        return params[o:o + int(np.prod(s))].reshape(s)

    part("tables")[:] = np.abs(part("tables")) + 0.5
    part("W1")[7], part("b1")[7] = -4.0, 1.0        # z1 = 1 - 4 sum(e) < 0 at every texel, 1 where e = 0
    part("W2")[11, :] = 0.0
    part("b2")[11] = 1.0
    want_p = params.copy()
    part("W2")[11, 7] = np.inf                       # inf * 0: this unit's sum is NaN, and the unit off
    gt = np.random.default_rng(44).uniform(-1, 1, (h, w, 4)).astype(np.float32)
    say("[gpu] ngp texels outside the texture")
    grads = []
    for p in (want_p, params):
        if p is want_p:
            o, s = lay["b2"]
            p[o + 11] = -1.0                         # the same unit off by its bias
        dev, ws = [torch.from_numpy(p).cuda()], P.ngp_workspace(cfg, [(w, h)])
        tex = P.ngp_bake(dev, cfg, [(w, h)], ws=ws)
        grads.append(P.ngp_backward(dev, cfg, [(w, h)], tex, [torch.from_numpy(gt).cuda()], ws)[0].cpu().numpy())
    assert np.isfinite(grads[1]).all()
    assert np.abs(grads[1] - grads[0]).max() <= GRAD_RTOL * np.abs(grads[0]).max()
