"""Two-level binning where it is taken (every case asserts that, by the workspace's block entries): plain bins
against a stable library sort of the duplicated entries, culled ones against the oracle's culled lists and
against the direct binning (the same scene by device counts with a capacity of 2^22, where the rule takes
the direct path, and of 2^22 + 1, where it takes the blocks); blocks of one entry up to tens of chunks of 512,
and a list of more chunks than the expansion's grids have workgroups."""
import numpy as np
import pytest

from oracle import oracle
from paper_2605_17855_amd import gs, scenes
from gpu_helpers import check_bins, note
from test_gpu_binning_route import bin_frame, same_bins

pytestmark = pytest.mark.gpu

DIRECT = 1 << 22


def _sorted_entries(b, cam, group):
    """Keys, Gaussians and masks of the footprints' entries, stably sorted by (bin, depth)."""
    gx = ((cam.width + 15) // 16 + group - 1) // group
    g = np.nonzero(b["count"])[0]
    x0, y0, x1, y1 = b["rect"][g].astype(np.int64).T
    bx0, by0 = x0 // group, y0 // group
    wd, ht = (x1 - 1) // group - bx0 + 1, (y1 - 1) // group - by0 + 1
    cnt = wd * ht
    i = np.repeat(np.arange(g.size), cnt)
    j = np.arange(i.size) - np.repeat(np.cumsum(cnt) - cnt, cnt)
    bx, by = bx0[i] + j % wd[i], by0[i] + j // wd[i]
    keys = ((by * gx + bx).astype(np.uint64) << np.uint64(32)) | b["depth"][g[i]].astype(np.uint64)
    mask = np.zeros(i.size, np.uint16)
    for ly in range(group):
        for lx in range(group):
            x, y = bx * group + lx, by * group + ly
            mask |= (((x0[i] <= x) & (x < x1[i]) & (y0[i] <= y) & (y < y1[i])).astype(np.uint16) << (ly * group + lx)).astype(np.uint16)
    order = np.argsort(keys, kind="stable")
    return keys[order], g[i][order].astype(np.uint32), mask[order]


def _check_ranges(b, k):
    bins = (b["keys"] >> np.uint64(32)).astype(np.int64)
    nb = b["ranges"].shape[0]
    start, end = np.searchsorted(bins, np.arange(nb)), np.searchsorted(bins, np.arange(nb), side="right")
    empty = start == end
    start[empty] = end[empty] = 0
    assert np.array_equal(b["ranges"], np.stack([start, end], 1))
    assert int((b["ranges"][:, 1].astype(np.int64) - b["ranges"][:, 0]).sum()) == k


# few splats over all tiles, many small ones, ragged, wide and tall grids; 9-bit bins (group 4 at 1080p),
# 9-bit blocks (2160p), few blocks of many entries
PLAIN = [(1, 300, 2560, 1440, 2.0), (1, 60000, 1281, 700, 0.02), (1, 20000, 3840, 2160, 0.03), (1, 9000, 530, 300, 0.3),
         (2, 1500, 1920, 1080, 1.0), (2, 40000, 3838, 2130, 0.05), (2, 30000, 4096, 129, 0.2),
         (4, 2500, 1920, 1080, 2.0), (4, 60000, 3840, 2160, 0.06), (4, 20000, 2049, 1100, 0.15), (1, 30000, 200, 4000, 0.2)]


@pytest.mark.parametrize("group,n,w,h,scale", PLAIN)
def test_plain_bins(group, n, w, h, scale):
    note(f"blocks coverage: n {n}, {w}x{h}, scale {scale}, group {group}")
    sc = scenes.camera_box_scene(n, seed=n, log_scale_mu=float(np.log(scale)))
    sc.mean[2, : n // 3] = sc.mean[2, 0]          # equal depths: ties in index order
    ds, cam = gs.DeviceScene(sc), scenes.pinhole(w, h, 60.0)
    k, blocks, b = bin_frame(ds, cam, group, False, 1 << 25)
    assert k >= 1 << 20 and blocks is not None and 0 < blocks <= k
    keys, vals, masks = _sorted_entries(b, cam, group)
    assert keys.size == k and np.array_equal(b["keys"], keys) and np.array_equal(b["vals"], vals)
    if group > 1:
        assert np.array_equal(b["masks"], masks)
    _check_ranges(b, k)


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("n,w,h,scale,opacity", [(2000, 2560, 1440, 0.2, 1.0), (9000, 2304, 1300, 0.08, 0.3)])
def test_culled_bins_against_the_oracle(n, w, h, scale, opacity, group):
    import torch
    note(f"blocks coverage, culled: n {n}, {w}x{h}, scale {scale}, group {group}")
    sc = scenes.camera_box_scene(n, seed=n, log_scale_mu=float(np.log(scale)))
    sc.opacity[::2] *= opacity
    sc.opacity[::7] = 0.003                        # below the cut: no entry
    cam = scenes.pinhole(w, h, 60.0)
    r = gs.Renderer(n, w, h, group=group, capacity=DIRECT + 1)
    opt = gs.options(group=group, precision="fp16", tight=True, device_counts=True)
    ds = gs.DeviceScene(sc)
    r.render(ds, cam, opt)
    torch.cuda.synchronize()
    k = gs.entry_count(r.proj)
    assert 0 < k <= DIRECT + 1
    check_bins(oracle.preprocess(sc, cam), cam, r, k, group, tight=True)
    assert bin_frame(ds, cam, group, True, DIRECT + 1, True)[1] is not None


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("n,w,h,scale,sigma", [(3_000_000, 2560, 1440, 0.0004, 0.3),   # more than 4,096 chunks
                                               (200_000, 2304, 1300, 0.006, 0.8),
                                               (6000, 3840, 2160, 0.01, 1.2),          # a few across the frame
                                               (700, 2560, 1440, 0.2, 0.8)])
def test_culled_bins_against_the_direct_path(n, w, h, scale, sigma, group):
    note(f"blocks coverage, culled by both paths: n {n}, {w}x{h}, scale {scale}, group {group}")
    sc = scenes.camera_box_scene(n, seed=n + 1, log_scale_mu=float(np.log(scale)), log_scale_sigma=sigma)
    sc.opacity[::2] *= 0.05
    ds, cam = gs.DeviceScene(sc), scenes.pinhole(w, h, 60.0)
    k, blocks, want = bin_frame(ds, cam, group, True, DIRECT, True)
    assert 0 < k <= DIRECT and blocks is None
    k2, blocks2, got = bin_frame(ds, cam, group, True, DIRECT + 1, True)
    assert k2 == k and blocks2 is not None and 0 < blocks2 <= k
    if n == 3_000_000:
        assert blocks2 > 4096 * 512
    same_bins(got, want, group)
    _check_ranges(got, k)
