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
