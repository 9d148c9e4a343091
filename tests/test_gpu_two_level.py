"""Two-level binning (8x8-tile blocks, then the bins inside them): ranges, indices, 64-bit keys
and membership masks equal to a stable library sort of the duplicated entries, made here on the
CPU from the same footprints, over grids around the block edges, one block and many, and list
lengths around the chunks.  (Opacity-aware bins are held to the oracle's culled lists by
test_gpu_tight; here their lists are the subset of the full lists that the masks of the
same scene with larger groups allow.)"""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu


def _bins(sc, cam, group, tight, device_counts=False):
    import torch
    ds = gs.DeviceScene(sc)
    r = gs.Renderer(sc.n, cam.width, cam.height, group=group, capacity=(1 << 22) + 1)   # (the path is chosen by it)
    r.render(ds, cam, gs.options(group=group, precision="fp16", tight=tight))
    if device_counts:
        r.bins.ranges.fill_(-1)
        r.render(ds, cam, gs.options(group=group, precision="fp16", tight=tight, device_counts=True))
    torch.cuda.synchronize()
    k = gs.entry_count(r.proj)
    u = lambda t, d: t.cpu().numpy().view(d)
    p = r.proj
    return dict(k=k, keys=u(r.bins.keys, np.uint64)[:k], vals=u(r.bins.vals, np.uint32)[:k],
                masks=u(r.bins.masks, np.uint16)[:k], ranges=u(r.bins.ranges, np.uint32),
                rect=u(p.rect, np.uint16), count=u(p.count, np.uint32), depth=u(p.rgb, np.uint32)[:, 3])


def _want(b, cam, group):
    """The same from the footprints: entries in index order, a stable sort by (bin, depth)."""
    tx = (cam.width + 15) // 16
    gx = (tx + group - 1) // group
    bins, vals, masks = [], [], []
    for g in np.nonzero(b["count"])[0]:
        x0, y0, x1, y1 = (int(v) for v in b["rect"][g])
        for by in range(y0 // group, (y1 - 1) // group + 1):
            for bx in range(x0 // group, (x1 - 1) // group + 1):
                m = 0
                for ly in range(group):
                    for lx in range(group):
                        if x0 <= bx * group + lx < x1 and y0 <= by * group + ly < y1:
                            m |= 1 << (ly * group + lx)
                bins.append(by * gx + bx)
                vals.append(g)
                masks.append(m)
    bins, vals = np.array(bins, np.uint64), np.array(vals, np.uint32)
    keys = (bins << np.uint64(32)) | b["depth"][vals].astype(np.uint64)
    order = np.argsort(keys, kind="stable")
    return keys[order], vals[order], np.array(masks, np.uint16)[order]


CASES = [  # n, width, height, scale: more than 256 bins at 4x4 groups down to single tiles (fewer take the
    # plain passes), grids of 6 up to 512 blocks, ragged, wide and tall
    (2, 272, 256, 0.3), (700, 530, 272, 0.1), (40, 1281, 1100, 1.0), (3000, 4096, 129, 0.05), (600, 1050, 1024, 2.0),
    (5000, 600, 400, 0.02), (1500, 3840, 2160, 0.03), (2000, 200, 4000, 0.05)]


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("n,w,h,scale", CASES)
def test_bins_match_a_library_sort(n, w, h, scale, group):
    note(f"two-level bins: n {n}, {w}x{h}, scale {scale}, group {group}")
    sc = scenes.camera_box_scene(n, seed=n, log_scale_mu=float(np.log(scale)))
    sc.mean[2, : n // 3] = sc.mean[2, 0]          # equal depths: ties in index order
    cam = scenes.pinhole(w, h, 60.0)
    for dev in (False, True):
        b = _bins(sc, cam, group, False, dev)
        keys, vals, masks = _want(b, cam, group)
        assert b["k"] == keys.size
        assert np.array_equal(b["keys"], keys) and np.array_equal(b["vals"], vals)
        if group > 1:
            assert np.array_equal(b["masks"], masks)
        bins = (keys >> np.uint64(32)).astype(np.int64)
        nb = b["ranges"].shape[0]
        start, end = np.searchsorted(bins, np.arange(nb)), np.searchsorted(bins, np.arange(nb), side="right")
        empty = start == end
        start[empty] = end[empty] = 0
        assert np.array_equal(b["ranges"], np.stack([start, end], 1))


@pytest.mark.parametrize("n,w,h,scale", CASES)
def test_culled_lists_agree_across_groups(n, w, h, scale):
    note(f"two-level culled bins: n {n}, {w}x{h}, scale {scale}")
    sc = scenes.camera_box_scene(n, seed=n + 1, log_scale_mu=float(np.log(scale)))
    sc.opacity[::2] *= 0.05
    cam = scenes.pinhole(w, h, 60.0)
    tx, ty = (w + 15) // 16, (h + 15) // 16
    tiles = {}
    for group in (1, 2, 4):
        b = _bins(sc, cam, group, True, group == 2)
        gx = (tx + group - 1) // group
        lists = []
        for t in range(tx * ty):
            x, y = t % tx, t // tx
            s, e = b["ranges"][(y // group) * gx + x // group]
            v, k = b["vals"][s:e], b["keys"][s:e] & np.uint64(0xFFFFFFFF)
            if group > 1:
                on = (b["masks"][s:e] >> ((y % group) * group + x % group)) & 1 != 0
                v, k = v[on], k[on]
            assert np.array_equal(k, np.sort(k, kind="stable"))
            lists.append(v)
        if group > 1:
            assert (b["masks"] != 0).all()
        tiles[group] = lists
        assert b["k"] == int(b["count"].sum())
    for t in range(tx * ty):
        assert np.array_equal(tiles[1][t], tiles[2][t]) and np.array_equal(tiles[1][t], tiles[4][t])
