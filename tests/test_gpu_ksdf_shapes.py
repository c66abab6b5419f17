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
