"""GPU raster at the edges of its triangle paths: chunk sizes at which a triangle's lanes change, boxes next to the
one-lane limit, large triangles, and more of them in one bin than its queue holds.  Visibility bit-exact against the
oracle, fragment counts equal."""
import numpy as np
import pytest

import oracle as O
import scenes as S
from vs_testlib import assert_vis_equal, gpu_render, say, vis_numpy

pytestmark = pytest.mark.gpu


def _soup(seed, n, boxes, size):
    """n triangles of both windings at random depths whose screen boxes are about the given pixel sizes."""
    rng = np.random.default_rng([91, seed, n])
    w, h = size
    cam = S.make_camera(w, h, (0.0, 0.0, 3.0))
    box = np.asarray(boxes, float)[rng.integers(0, len(boxes), n)]
    at = rng.uniform([0.0, 0.0], [max(w - 1, 1), max(h - 1, 1)], (n, 2)) - box * rng.uniform(0.2, 0.8, (n, 1))
    corner = rng.uniform(0.0, 1.0, (n, 3, 2))
    corner[:, 0, 0], corner[:, 1, 1], corner[:, 2] = 0.0, 0.0, 1.0   # the box's extents are met
    flip = rng.random(n) < 0.5
    corner[flip] = corner[flip][:, [0, 2, 1]]
    px = at[:, None, :] + corner * box[:, None, :]
    z = rng.uniform(1.0, 4.0, (n, 1)) * rng.uniform(0.9, 1.1, (n, 3))
    p = np.stack([(px[..., 0] - cam.cx) / cam.fx * z, (px[..., 1] - cam.cy) / cam.fy * z, z], -1)
    xyz = (p.reshape(-1, 3) - cam.t) @ cam.R   # R^T (p - t)
    uv = rng.uniform(0.0, 1.0, (3 * n, 2))
    mesh = S.Mesh(xyz.astype(np.float32), uv.astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3))
    tex = [S.uniform_texture(91, 0, 8, 8, opaque=True)]
    return S.Scene(f"soup{n}", [mesh], tex, [cam])


SMALL, EDGE, LARGE = [(3, 3), (9, 5)], [(22, 22), (32, 15), (26, 18), (63, 7), (64, 8)], [(66, 10), (40, 40), (200, 150)]


@pytest.mark.parametrize("bin", [8, 16, 32, 64])
@pytest.mark.parametrize("n,boxes,size", [
    (1, EDGE, (64, 56)), (16, EDGE, (64, 56)), (17, EDGE, (64, 56)), (33, EDGE, (61, 53)), (65, SMALL, (64, 56)),
    (128, SMALL, (64, 56)), (129, EDGE, (64, 56)), (256, SMALL, (64, 56)), (300, SMALL + EDGE, (64, 56)),
    (5, LARGE, (201, 133)), (192, LARGE, (64, 56)), (500, LARGE, (64, 56)), (700, SMALL + EDGE + LARGE, (201, 133))])
def test_triangle_paths(bin, n, boxes, size):
    import torch
    assert torch.cuda.is_available()
    sc = _soup(len(boxes), n, boxes, size)
    want, ref = O.raster(sc.layers[0], sc.cameras[0])
    assert (want != np.uint64(0xFFFFFFFFFFFFFFFF)).any()
    for count in (False, True):
        say(f"[gpu] soup n={n} {size} bin {bin} count {count}")
        P, layers, views, vis, ws, _, _ = gpu_render(sc, bin=bin, count_fragments=count)
        assert_vis_equal(vis_numpy(views, vis, 1, 0)[0][None], want[None], f"n={n} bin {bin}")
        if count:
            assert P.read_status(ws)["fragments"] == ref["fragments"]


def _check(sc, what, **kw):
    for count in (False, True):
        say(f"[gpu] {what} count {count}")
        P, layers, views, vis, ws, _, _ = gpu_render(sc, count_fragments=count, **kw)
        frags = 0
        for v, cam in enumerate(sc.cameras):
            for l, m in enumerate(sc.layers):
                want, ref = O.raster(m, cam)
                frags += ref["fragments"]
                assert_vis_equal(vis_numpy(views, vis, sc.k, v)[l][None], want[None], f"{what} view {v} layer {l}")
        st = P.read_status(ws)
        assert not count or st["fragments"] == frags
    return st


def _shuffled(k, n_lat, n_lon, sizes):
    """Displaced shells whose triangles come in random order: every group of consecutive ones reaches every tile."""
    rng = np.random.default_rng([92, k, n_lat])
    layers = [S.Mesh(m.xyz, m.uv, m.tri[rng.permutation(m.n_tri)]) for m in S.displaced_shells(2, k, n_lat, n_lon)]
    tex = [S.uniform_texture(92, l, 8, 8, opaque=True) for l in range(k)]
    return S.Scene("shuffled", layers, tex, S.ring_cameras(92, len(sizes), sizes))


@pytest.mark.parametrize("bin", [16, 64])
@pytest.mark.parametrize("k,n_lat,n_lon,sizes", [
    (2, 160, 320, [(300, 200)]),        # 398 groups of 256 triangles a layer, all in the middle bins: loaded in turns
    (4, 160, 321, [(120, 90)]),         # groups of 512
    (1, 160, 320, [(61, 40)] * 21),     # groups of 1,024
    (1, 5, 32, [(70, 70)]),             # exactly 256 triangles: one full group
])
def test_groups_in_random_order(bin, k, n_lat, n_lon, sizes):
    _check(_shuffled(k, n_lat, n_lon, sizes), f"shuffled k={k} {n_lat}x{n_lon} {len(sizes)} views bin {bin}", bin=bin)


@pytest.mark.parametrize("boxes", [SMALL, LARGE])
def test_groups_over_more_tiles_than_a_table_holds(boxes):
    """1,024 x 9 bins of 8 pixels under one group: its table counts 2 x 2 bins at a time."""
    _check(_soup(7, 700, boxes, (8192, 72)), f"wide {len(boxes)}", bin=8)


@pytest.mark.parametrize("capacity", [1, 600, 4000, 20000])
def test_groups_without_list_space(capacity):
    """Groups that find no room in the list are gone through triangle by triangle, next to groups that found some."""
    sc = _shuffled(2, 60, 120, [(200, 150), (90, 140)])
    assert _check(sc, f"capacity {capacity}", list_capacity=capacity)["bin_overflow"] > 0


@pytest.mark.parametrize("k,size", [(3, (256, 256)), (3, (640, 336)), (4, (512, 300)), (5, (600, 560)), (7, (900, 900))])
def test_library_choice_of_bin(k, size):
    """Calls that leave the bin to the library, on both sides of the counts at which it takes 16, 32 and 64 pixels: the
    visibility of every explicit size, in a workspace of the default's 64-pixel size."""
    import torch
    import paper_2409_02482_amd as P
    layers = P.Layers(S.displaced_shells(3, k, 20, 40))
    views = P.Views(S.ring_cameras(4, 1, [size]))
    assert P.workspace_bytes(layers, views) == P.workspace_bytes(layers, views, 64)
    vis, ws = P.raster(layers, views, count_fragments=True)
    st = P.read_status(ws)
    assert st["bin_overflow"] == 0
    for b in (16, 32, 64):
        other, ws2 = P.raster(layers, views, bin=b, count_fragments=True)
        assert torch.equal(vis, other) and P.read_status(ws2)["fragments"] == st["fragments"], b


@pytest.mark.parametrize("k,lat,lon,sizes", [
    (3, 20, 34, [(800, 800)] * 64),
    (1, 20, 34, [(800, 800)] * 100),
    (5, 20, 40, [(1600, 1080)] * 24),
    (7, 20, 34, [(96, 96)] * 40 + [(4096, 4096)] + [(96, 96)] * 23),
])
def test_coarse_shells_in_many_views(k, lat, lon, sizes):
    """Large triangles in many views, and one large view among small ones: the default workspace holds all their entries."""
    import torch
    import paper_2409_02482_amd as P
    say(f"[gpu] coarse shells k={k} {lat}x{lon} {len(sizes)} views")
    layers = P.Layers(S.displaced_shells(2, k, lat, lon))
    views = P.Views(S.ring_cameras(5, len(sizes), sizes))
    vis, ws = P.raster(layers, views)
    assert P.read_status(ws)["bin_overflow"] == 0
    direct, _ = P.raster(layers, views, direct=True)
    assert torch.equal(vis, direct)


@pytest.mark.parametrize("bin", [8, 32, 64])
@pytest.mark.parametrize("boxes,size", [(SMALL, (8192, 72)), (LARGE, (2048, 1100)), (SMALL + LARGE, (300, 5000))])
def test_depth_bounds_of_back_faces(bin, boxes, size):
    """Both windings over many depths, in macro tiles of one to several bins: a back face is skipped only where it cannot be
    seen.  Against the unbinned path, with and without the fragment count that skips nothing."""
    import torch
    import paper_2409_02482_amd as P
    sc = _soup(5, 3000, boxes, size)
    layers, views = P.Layers(sc.layers), P.Views(sc.cameras)
    say(f"[gpu] soup of 3000 {size} bin {bin}")
    direct, ws = P.raster(layers, views, direct=True, count_fragments=True)
    frags = P.read_status(ws)["fragments"]
    assert torch.equal(P.raster(layers, views, bin=bin)[0], direct)
    vis, ws = P.raster(layers, views, bin=bin, count_fragments=True)
    assert torch.equal(vis, direct) and P.read_status(ws)["fragments"] == frags


def test_capacity_is_a_count_of_pairs():
    """list_capacity counts (triangle, bin) pairs: as many as the scene has fit, one fewer does not."""
    from test_list_room import _boxes
    sc = _shuffled(2, 60, 120, [(200, 150), (90, 140)])
    b = _boxes(sc.layers, sc.cameras)
    b = b[b[:, 0] == 1]
    pairs = int(((b[:, 3] // 64 - b[:, 2] // 64 + 1) * (b[:, 5] // 56 - b[:, 4] // 56 + 1)).sum())
    assert _check(sc, "capacity of all pairs", list_capacity=pairs)["bin_overflow"] == 0
    assert _check(sc, "capacity one short", list_capacity=pairs - 1)["bin_overflow"] > 0


def test_more_entries_than_a_table_sums():
    """256 triangles over most of 992 bins each: more entries of a side than a table's 16-bit sums, in macro tiles then."""
    sc = _soup(6, 700, [(600, 600)], (256, 248))
    assert _check(sc, "wide soup", bin=8)["bin_overflow"] == 0


@pytest.mark.parametrize("k,n_lat,size,bin", [(1, 520, (1024, 1024), 16), (2, 400, (1100, 1030), 16), (1, 300, (512, 300), 32)])
def test_many_groups_in_random_order(k, n_lat, size, bin):
    """More groups with an entry or two in a bin than a block takes at once, and groups enlarged for a view of many tiles."""
    import torch
    import paper_2409_02482_amd as P
    say(f"[gpu] shuffled k={k} {n_lat}x{2 * n_lat} {size} bin {bin}")
    sc = _shuffled(k, n_lat, 2 * n_lat, [size])
    layers, views = P.Layers(sc.layers), P.Views(sc.cameras)
    direct, ws = P.raster(layers, views, direct=True, count_fragments=True)
    frags = P.read_status(ws)["fragments"]
    assert torch.equal(P.raster(layers, views, bin=bin)[0], direct)
    vis, ws = P.raster(layers, views, bin=bin, count_fragments=True)
    st = P.read_status(ws)
    assert torch.equal(vis, direct) and st["fragments"] == frags and st["bin_overflow"] == 0


@pytest.mark.parametrize("bin,capacity", [(64, 3000), (64, 300000), (16, 100000), (8, 1000000)])
def test_many_groups_at_once_without_list_space(bin, capacity):
    """Hundreds of groups ask for room at the same time and most find none: the others' runs stay theirs."""
    import torch
    import paper_2409_02482_amd as P
    say(f"[gpu] 24 views, bin {bin}, capacity {capacity}")
    layers = P.Layers(S.displaced_shells(2, 5, 40, 80))
    views = P.Views(S.ring_cameras(5, 24, [(640, 500)] * 24))
    vis, ws = P.raster(layers, views, bin=bin, list_capacity=capacity)
    assert P.read_status(ws)["bin_overflow"] > 0
    assert torch.equal(vis, P.raster(layers, views, direct=True)[0])
