"""k-SDF rendering at the edges of its lane layouts, against the FP64 oracle.

A ray's march steps come in groups of 64 (64, 192, 320, 2048 steps: one group,
remainders of the groups of four, the most), its samples in one to four slots
of 32 with one to four samples a lane in each importance round (counts below,
at and above multiples of 32; a round of more than 32 new samples), and a
wavefront's rays in batches (odd totals, views that end inside a batch).
Without importance rounds every sample position is the oracle's bit for bit,
which needs every march step's voxel; colours and per-surface values within
1e-5, the bar of FP32 weights over FP64 samples (a few hundred roundings of
6e-8).  Rays along a voxel face have no unique result and are left out."""
import numpy as np
import pytest

import scenes as S
from oracle import ksdf as K
from test_gpu_ksdf import TOL, _setup, torch_cuda  # noqa: F401
from vs_testlib import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,n,m,steps,occ_res,sizes", [
    (1, 2, 0, 64, 1, [(5, 3)]),
    (3, 33, 0, 192, 37, [(17, 13), (1, 1), (7, 9)]),
    (2, 30, 6, 320, 40, [(31, 11)]),
    (3, 20, 100, 320, 33, [(13, 17), (19, 5)]),
    (4, 64, 64, 2048, 64, [(16, 16)]),
    (2, 97, 2, 64, 255, [(33, 7)]),
    (16, 32, 32, 256, 16, [(21, 9)]),
])
def test_ksdf_lane_layouts(torch_cuda, k, n, m, steps, occ_res, sizes):  # noqa: F811
    torch = torch_cuda
    g = S.ksdf_grids(71, 48, 24)
    P, field, opts, oopts = _setup(torch, g, k, occ_res, n_uniform=n, n_importance=m, march_steps=steps)
    cams = S.ring_cameras(72, len(sizes), sizes)
    occ_np = K.occupancy(g, oopts)
    occ = P.ksdf_occupancy(field, opts)
    rgba, lay, smp = P.ksdf_render(field, opts, occ, P.Views(cams), layers=True, samples=True)
    torch.cuda.synchronize()
    rgba, lay, smp = rgba.cpu().numpy(), lay.cpu().numpy(), smp.cpu().numpy()
    off = live = 0
    for cam in cams:
        want = K.render(g, oopts, occ_np, cam)
        sl = slice(off, off + cam.width * cam.height)
        off = sl.stop
        o, d = K.camera_rays(cam)
        keep = ~K.march_on_face(o, d, oopts.occ_res, g.lo, g.hi, oopts.march_steps)
        empty = want["samples"][:, 0] < 0
        live += int((~empty & keep).sum())
        err, lerr = np.abs(rgba[sl] - want["rgba"])[keep], np.abs(lay[:, sl] - want["layers"])[:, keep]
        say(f"[gpu] ksdf lanes n={n} m={m} steps={steps}: colour err {err.max(initial=0):.2e}, "
            f"layer err {lerr.max(initial=0):.2e}, {int((~keep).sum())} rays left out")
        assert np.array_equal(smp[sl, 0][keep] < 0, empty[keep])
        assert err.max(initial=0) <= TOL and lerr.max(initial=0) <= TOL
        if m == 0:
            assert np.array_equal(smp[sl][keep], want["samples"][keep])
        else:
            gap = np.diff(want["samples"], axis=1).max(1)
            assert (np.abs(smp[sl] - want["samples"]).max(1) <= np.maximum(gap, 0.0))[~empty & keep].all()
    assert live > 0


def _positions_at(t, d, offsets, beta, u, eps):
    """Parameters at CDF values u [m] (clipped to 0..1) of one importance round over samples t, d [rays, N]."""
    W = sum(K.neus_weights(d, o, beta) for o in offsets) + eps
    cdf = np.concatenate([np.zeros((len(t), 1)), np.cumsum(W, 1) / W.sum(1, keepdims=True)], 1)
    u = np.clip(u, 0.0, 1.0)
    return np.stack([np.interp(u, cdf[r], t[r]) for r in range(len(t))])


@pytest.mark.parametrize("k,n,m,steps,occ_res,sizes", [
    (3, 20, 100, 320, 33, [(13, 17), (19, 5)]),
    (2, 30, 6, 320, 40, [(31, 11)]),
    (4, 64, 64, 2048, 64, [(16, 16)]),
    (2, 97, 2, 64, 255, [(33, 7)]),
    (7, 64, 32, 1024, 64, [(24, 20)]),
    (16, 32, 32, 256, 16, [(21, 9)]),
])
def test_ksdf_merged_samples(torch_cuda, k, n, m, steps, occ_res, sizes):  # noqa: F811
    """The merged list of a ray: in order, the uniform samples among it bit for bit, and each importance sample where the
    oracle's CDF puts it within 1e-3 (a twentieth and less of the distance to the next sample, and a hundred times what FP32
    weights move it)."""
    torch = torch_cuda
    g = S.ksdf_grids(71, 48, 24)
    P, field, opts, oopts = _setup(torch, g, k, occ_res, n_uniform=n, n_importance=m, march_steps=steps)
    _, _, uniform, _ = _setup(torch, g, k, occ_res, n_uniform=n, n_importance=0, march_steps=steps)
    cams = S.ring_cameras(72, len(sizes), sizes)
    occ = P.ksdf_occupancy(field, opts)
    views = P.Views(cams)
    say(f"[gpu] ksdf merge n={n} m={m} steps={steps}")
    got = P.ksdf_render(field, opts, occ, views, samples=True)[-1].cpu().numpy()
    base = P.ksdf_render(field, uniform, occ, views, samples=True)[-1].cpu().numpy()
    o, v = (np.concatenate(x) for x in zip(*[K.camera_rays(c) for c in cams]))
    live = (base[:, 0] >= 0) & ~K.march_on_face(o, v, oopts.occ_res, g.lo, g.hi, oopts.march_steps)
    got, base, o, v = got[live], base[live], o[live], v[live]
    assert live.sum() > 20 and (np.diff(got, axis=1) >= 0).all()
    new = np.empty((len(got), m))
    for r in range(len(got)):
        rest = list(got[r])
        for t in base[r]:
            rest.remove(t)      # raises if it is not there
        new[r] = rest

    def sdf_along(tt):
        return K.sdf_at(g, (o[:, None, :] + tt[..., None] * v[:, None, :]).reshape(-1, 3)).reshape(tt.shape)

    t, d = base, sdf_along(base)
    u = (np.arange(m // 2) + 0.5) / (m // 2)
    bounds = [[], []]
    for beta in (oopts.beta / 2.0, oopts.beta):
        for side, delta in enumerate((-1e-3, 1e-3)):
            bounds[side].append(_positions_at(t, d, oopts.offsets, beta, u + delta, oopts.pdf_floor))
        tn = K.importance_round(t, d, oopts.offsets, beta, m // 2, oopts.pdf_floor)
        t, d = K.merge_sorted(t, d, tn, sdf_along(tn))
    low, high = (np.sort(np.concatenate(b, 1), 1) for b in bounds)
    assert (new >= low - 1e-12).all() and (new <= high + 1e-12).all()
