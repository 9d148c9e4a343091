"""Which frames are binned by way of 8x8-tile blocks: by their own entries, not by the room there is for
them (a pool's capacity, a larger earlier frame).  The path shows in the workspace's last words, where the
binning by blocks leaves the number of its block entries.  Both paths' bins are equal, so a scene's bins
are the same whatever the capacity."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu

COUNTS = 256         # the workspace ends with a block of this size: K, V, K clamped, block entries
UNTOUCHED = 0x7E7E7E7E


def bin_frame(ds, cam, group, tight, capacity, device_counts=False):
    """Bins one frame; returns (entries, block entries or None for the direct path, bins)."""
    import torch
    r = gs.Renderer(ds.n, cam.width, cam.height, group=group, capacity=capacity)
    opt = gs.options(group=group, precision="fp16", tight=tight, device_counts=device_counts)
    r.ws.fill_(0x7E)
    gs.gs_preprocess(ds, cam, opt, r.proj, r.ws)
    gs.gs_bin_sort(r.proj, cam, opt, r.bins, r.ws)
    torch.cuda.synchronize()
    k = gs.entry_count(r.proj)
    blocks = int(r.ws[-COUNTS:].view(torch.int32)[6].item()) & 0xFFFFFFFF
    u = lambda t, d: t.cpu().numpy().view(d)
    return k, None if blocks == UNTOUCHED else blocks, dict(
        keys=u(r.bins.keys, np.uint64)[:k], vals=u(r.bins.vals, np.uint32)[:k],
        masks=u(r.bins.masks, np.uint16)[:k], ranges=u(r.bins.ranges, np.uint32),
        rect=u(r.proj.rect, np.uint16), count=u(r.proj.count, np.uint32), depth=u(r.proj.rgb, np.uint32)[:, 3])


def same_bins(a, b, group):
    for f in ("keys", "vals", "ranges") + (("masks",) if group > 1 else ()):
        assert np.array_equal(a[f], b[f]), f


def scene(n, scale, seed, sigma=0.5):
    return gs.DeviceScene(scenes.camera_box_scene(n, seed=seed, log_scale_mu=float(np.log(scale)), log_scale_sigma=sigma))


@pytest.mark.parametrize("n", [3000, 40000])     # the one-launch depth sort and the passes
@pytest.mark.parametrize("group", [1, 2, 4])
def test_room_alone_changes_no_route(n, group):
    note(f"binning route: few entries, much room, n {n}, group {group}")
    ds, cam = scene(n, 0.02 if n < 8192 else 0.004, n), scenes.pinhole(2560, 1440, 60.0)
    k, blocks, bins = bin_frame(ds, cam, group, False, 1 << 20)
    assert k < 1 << 20 and blocks is None
    k2, blocks2, bins2 = bin_frame(ds, cam, group, False, 1 << 24)
    assert k2 == k and blocks2 is None
    same_bins(bins, bins2, group)


@pytest.mark.parametrize("n", [3000, 40000])
@pytest.mark.parametrize("tight", [False, True])
def test_many_entries_go_by_blocks(n, tight):
    note(f"binning route: many entries, n {n}, culled {tight}")
    ds, cam = scene(n, 0.1 if n < 8192 else 0.03, n), scenes.pinhole(2560, 1440, 60.0)
    k, blocks, bins = bin_frame(ds, cam, 1, tight, 1 << 25)
    assert k >= 1 << 20 and blocks is not None and 0 < blocks < k
    k2, blocks2, bins2 = bin_frame(ds, cam, 1, tight, k)     # (no room to spare)
    assert (k2, blocks2) == (k, blocks)
    same_bins(bins, bins2, 1)


def test_a_frame_without_entries():
    """Nothing visible: no bins on either path, also where the capacity chooses the blocks."""
    note("binning route: nothing visible")
    for n in (100, 20000):
        sc = scenes.camera_box_scene(n, seed=1)
        sc.mean[2] = -1.0
        ds, cam = gs.DeviceScene(sc), scenes.pinhole(2560, 1440, 60.0)
        for device_counts in (False, True):
            k, blocks, bins = bin_frame(ds, cam, 1, False, 1 << 23, device_counts)
            assert k == 0 and blocks == (0 if device_counts else None) and not bins["ranges"].any()
