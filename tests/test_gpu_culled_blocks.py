"""Two-level binning of long diagonal splats under opacity-aware culling with tile groups, where a
footprint overlaps far more 8x8-tile blocks than the ellipse meets bins: the same bins as the
direct binning, in a time of its order.  (Both by device counts, where the capacity chooses the
path.)  An entry's block was once looked for block by block over the whole footprint: five times the direct
binning's time on this scene, so twice is the bar for a path that takes less."""
import time

import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu

DIRECT = 1 << 22   # the largest capacity of the direct path under culling


def _scene():
    """500 splats, long (up to hundreds of pixels) and thin."""
    return scenes.camera_box_scene(500, seed=3, log_scale_mu=float(np.log(0.66)), log_scale_sigma=0.5)


def _bin(ds, cam, group, capacity):
    import torch
    r = gs.Renderer(ds.n, cam.width, cam.height, group=group, capacity=capacity)
    opt = gs.options(group=group, precision="fp16", tight=True, device_counts=True)
    gs.gs_preprocess(ds, cam, opt, r.proj, r.ws)
    best = float("inf")
    for _ in range(12):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(5):
            gs.gs_bin_sort(r.proj, cam, opt, r.bins, r.ws)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 5)
    k = gs.entry_count(r.proj)
    return best, k, [t.cpu().numpy() for t in (r.bins.keys[:k], r.bins.vals[:k], r.bins.masks[:k], r.bins.ranges)]


@pytest.mark.parametrize("group", [2, 4])
def test_long_splats(group):
    note(f"culled blocks: long splats, group {group}")
    ds, cam = gs.DeviceScene(_scene()), scenes.pinhole(3840, 2160, 60.0)
    direct, k, want = _bin(ds, cam, group, DIRECT)
    blocks, k2, got = _bin(ds, cam, group, DIRECT + 1)
    print(f"group {group}: {k} entries, direct {direct * 1e6:.0f} us, by blocks {blocks * 1e6:.0f} us")
    assert k == k2 and 100_000 < k < DIRECT
    for a, b in zip(want, got):
        assert np.array_equal(a, b)
    assert blocks <= 2 * direct
