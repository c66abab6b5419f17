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


def _everywhere(torch, P, field, opts):
    return P.ksdf_occupancy(field, opts).fill_(-1)


def _at_samples(g, oopts, o, v, t):
    """Layers [k, rays, 4] in 64 bits at the samples t that a render took (FP32 importance weights need not put them where
    the oracle's would), and how many ends of intervals lie where the plain quotient does not hold.  Next to a NaN the opacity
    is 0, but 1 from a NaN to a point so far inside that Phi is 0 in FP32 (that of the main surface, where offsets are a
    factor); it is 0 from and 1 to a point where Phi is 0 in FP64."""
    out, odd = [], 0
    factor = all(abs(oopts.beta * off) <= 60.0 for off in oopts.offsets)
    p = (o[:, None, :] + t[..., None] * v[:, None, :]).reshape(-1, 3)
    with np.errstate(all="ignore"):
        d = K.sdf_at(g, p).reshape(t.shape)
        app = K.rgba_at(g, p).reshape(*t.shape, 4)[:, :-1]
        nrm = K.sdf_normals(g, p).reshape(*t.shape, 3)[:, :-1]
        vdn = np.nan_to_num(np.abs((nrm * v[:, None, :]).sum(-1)), nan=0.0)
        aw = (2.0 / (1.0 + np.exp(-10.0 * vdn)) - 1.0) * app[..., 3]
        for off in oopts.offsets:
            x, y = -oopts.beta * (d[:, :-1] + off), -oopts.beta * (d[:, 1:] + off)
            phi, nxt = 1.0 / (1.0 + np.exp(x)), 1.0 / (1.0 + np.exp(y))
            a = np.where(phi > 0, np.maximum((phi - nxt) / phi, 0.0), 0.0)
            a = np.where(np.isnan(x) | np.isnan(y), 0.0, a)
            inside = np.float32(-oopts.beta * (d[:, 1:] + (0.0 if factor else off)))
            a = np.where(np.isnan(x) & (np.isinf(np.exp(inside)) | (y > 709.79)), 1.0, a)
            odd += int((np.isnan(x) | (x > 709.0)).sum())
            w = np.cumprod(np.concatenate([np.ones((len(a), 1)), 1.0 - a[:, :-1]], 1), 1) * a
            out.append(np.concatenate([(w[..., None] * app[..., :3]).sum(1), (w * aw).sum(1)[:, None]], 1))
    return np.stack(out), odd


def _check_layers(lay, want):
    """Colours of all rays; opacities of all but the few rays that run along a cell face, where the normal jumps."""
    err = np.abs(lay - want)
    assert err[..., :3].max() <= TOL, err[..., :3].max()
    assert (err[..., 3] > TOL).mean() <= 0.002, err[..., 3].max()


@pytest.mark.parametrize("k,offsets,far,n,m", [
    (1, [0.0], 0.25, 64, 32), (4, [-0.3, 0.0, 0.1, 0.4], 0.25, 64, 64), (3, None, 0.3, 33, 6), (16, None, 0.2, 16, 8)])
def test_ksdf_from_far_inside(torch_cuda, k, offsets, far, n, m):  # noqa: F811
    """A camera near the middle of the object, every voxel taken for occupied: where Phi is 0 in FP64 there is no opacity,
    however the distance falls along the ray."""
    torch = torch_cuda
    g = S.ksdf_grids(71, 48, 24)
    P, field, opts, oopts = _setup(torch, g, k, 64, offsets=offsets, n_uniform=n, n_importance=m, march_steps=512)
    cams = S.ring_cameras(72, 2, [(31, 20), (16, 24)], far)
    say(f"[gpu] ksdf from inside k={k} far={far}")
    got, lay, smp = (x.cpu().numpy() for x in P.ksdf_render(field, opts, _everywhere(torch, P, field, opts), P.Views(cams),
                                                           layers=True, samples=True))
    o, v = (np.concatenate(x) for x in zip(*[K.camera_rays(c) for c in cams]))
    want, odd = _at_samples(g, oopts, o, v, smp)
    assert odd > 50
    _check_layers(lay, want)
    col, T = np.zeros((len(o), 3)), np.ones(len(o))
    for C in lay.astype(np.float64):
        col += (T * C[:, 3])[:, None] * C[:, :3]
        T *= 1.0 - C[:, 3]
    assert np.abs(got - np.concatenate([col, 1.0 - T[:, None]], 1)).max() <= TOL


@pytest.mark.parametrize("bad", [np.nan, -np.inf, -1e30, 1e30])
@pytest.mark.parametrize("k,offsets,n,m", [(3, None, 33, 6), (4, [-0.3, 0.0, 0.1, 0.4], 64, 64), (7, None, 64, 32)])
def test_ksdf_fields_with_odd_values(torch_cuda, bad, k, offsets, n, m):  # noqa: F811
    """Infinite, huge and NaN values in the distance grid."""
    torch = torch_cuda
    g = S.ksdf_grids(71, 48, 24)
    g.sdf.reshape(-1)[np.random.default_rng([73, k]).integers(0, g.sdf.size, 400)] = bad
    P, field, opts, oopts = _setup(torch, g, k, 64, offsets=offsets, n_uniform=n, n_importance=m, march_steps=512)
    cam = S.ring_cameras(72, 1, [(48, 40)], 2.0)[0]
    say(f"[gpu] ksdf fields with {bad} k={k}")
    _, lay, smp = (x.cpu().numpy() for x in P.ksdf_render(field, opts, _everywhere(torch, P, field, opts), P.Views([cam]),
                                                         layers=True, samples=True))
    o, v = K.camera_rays(cam)
    live = (smp[:, 0] >= 0) & np.isfinite(smp).all(1)
    want, odd = _at_samples(g, oopts, o[live], v[live], smp[live])
    assert live.sum() > 500 and (bad > 0 or odd > 100)
    _check_layers(lay[:, live], want)
