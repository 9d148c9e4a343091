"""The FP32 rasterizer of whole 2x2 groups, which large culled frames take: image and every auxiliary
plane bit-identical to the member-tile rasterizer over the same bins (the one the same bins get without
GS_OPT_TIGHT among the rasterizer's options), on one image, in a batch of equal images and in a
batch whose smaller image keeps all jobs to the member tiles; and no slower on the dense scene, where
the row reads of four workgroups per group took 1.4 times as long."""
import time

import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note
from test_gpu_fp32_lists import AUX

pytestmark = pytest.mark.gpu


def _frame(sc, cam, group):
    r = gs.Renderer(sc.n, cam.width, cam.height, group=group)
    r.render(gs.DeviceScene(sc), cam, _opt(group, True))
    return r


def _opt(group, tight, aux=0):
    return gs.options(group=group, precision="fp32", bg=(0.3, 0.2, 0.1), tight=tight, aux_flags=aux)


def _raster(r, cam, opt):
    import torch
    image = torch.zeros_like(r.image)
    aux = torch.zeros((5, cam.height, cam.width), dtype=torch.float32, device="cuda") if opt.aux_flags else None
    gs.gs_rasterize(r.proj, r.bins, cam, opt, image, aux)
    torch.cuda.synchronize()
    return image, aux


def _batch(frames, opt):
    import torch
    ctr = torch.zeros(gs.BATCH_COUNTER_WORDS, dtype=torch.int32, device="cuda")
    out = [torch.zeros_like(r.image) for r, _ in frames]
    gs.gs_rasterize_batch([(r.proj, r.bins, cam, o, None) for (r, cam), o in zip(frames, out)], opt, ctr)
    torch.cuda.synchronize()
    return out


# 7,168 groups are 112 x 64; ragged sizes, lists of less than a chunk up to several
@pytest.mark.parametrize("n,w,h,scale", [(60, 3584, 2048, 0.5), (2000, 3571, 2039, 0.2), (30000, 3605, 2050, 0.03)])
def test_whole_groups_match_member_tiles(n, w, h, scale):
    import torch
    note(f"fp32 whole groups: n {n}, {w}x{h}")
    sc = scenes.camera_box_scene(n, seed=n, log_scale_mu=float(np.log(scale)))
    sc.opacity[: n // 2] *= 0.2
    cam = scenes.pinhole(w, h, 60.0)
    r = _frame(sc, cam, 2)
    image, aux = _raster(r, cam, _opt(2, True, AUX))
    want, waux = _raster(r, cam, _opt(2, False, AUX))
    assert torch.equal(image, want) and torch.equal(aux, waux)
    plain, _ = _raster(r, cam, _opt(2, True))          # (the kernel without the planes)
    assert torch.equal(plain, want)
    small = scenes.pinhole(640, 360, 60.0)
    rs = _frame(sc, small, 2)
    swant, _ = _raster(rs, small, _opt(2, False))
    for frames, expect in (([(r, cam), (r, cam)], [want, want]), ([(r, cam), (rs, small)], [want, swant])):
        for a, b in zip(_batch(frames, _opt(2, True)), expect):
            assert torch.equal(a, b)


def test_dense_frame_is_faster_by_whole_groups():
    import torch
    sc = scenes.camera_box_scene(300_000, seed=4, log_scale_mu=float(np.log(0.05)))
    note("fp32 whole groups: dense frame at 3840x2160")
    cam = scenes.pinhole(3840, 2160, 60.0)
    r = _frame(sc, cam, 2)

    def best(opt):
        t = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                gs.gs_rasterize(r.proj, r.bins, cam, opt, r.image)
            torch.cuda.synchronize()
            t.append((time.perf_counter() - t0) / 5)
        return min(t)

    whole, tiles = best(_opt(2, True)), best(_opt(2, False))
    print(f"whole groups {whole * 1e6:.0f} us, member tiles {tiles * 1e6:.0f} us")
    assert whole <= 0.9 * tiles
