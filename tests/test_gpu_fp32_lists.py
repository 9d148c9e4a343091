"""The FP32 rasterizer's per-quadrant row lists and member-tile row buffer: every image and
auxiliary plane bit-identical to the one that runs every row in every quadrant
(GS_OPT_ALL_ROWS), for lists of one row up to several chunks and buffer fills, and for groups
equal to single tiles up to the FP32 rounding of the group-relative centres."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu

AUX = gs.GS_AUX_TFINAL | gs.GS_AUX_WSUM | gs.GS_AUX_NEVAL | gs.GS_AUX_NBLEND | gs.GS_AUX_LAST


def _render(sc, cam, group, all_rows):
    import torch
    ds = gs.DeviceScene(sc)
    r = gs.Renderer(sc.n, cam.width, cam.height, group=group, capacity=64 * sc.n + 1024)
    r.render(ds, cam, gs.options(group=group, precision="fp32", bg=(0.3, 0.2, 0.1), aux_flags=AUX, all_rows=all_rows))
    torch.cuda.synchronize()
    return r.image.cpu().numpy(), r.aux.cpu().numpy()


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("n,w,h,sigma", [(1, 16, 16, 0.02), (255, 17, 15, 0.3), (257, 33, 31, 0.3),
                                         (700, 70, 33, 0.3), (6000, 131, 77, 0.02)])
def test_row_lists_change_no_output(group, n, w, h, sigma):
    note(f"fp32 lists: n {n}, {w}x{h}, group {group}")
    sc = scenes.camera_box_scene(n, seed=n, log_scale_mu=float(np.log(sigma)))
    sc.opacity[: n // 2] *= 0.2           # long lists: few pixels stop early
    cam = scenes.pinhole(w, h, 60.0)
    img, aux = _render(sc, cam, group, False)
    img_all, aux_all = _render(sc, cam, group, True)
    assert np.array_equal(img, img_all) and np.array_equal(aux, aux_all)
    if group > 1:
        # the power's FP32 rounding differs with the frame of the centres: 1e-4 is the bar of
        # the FP32 image against the oracle, so twice that between two frames of it
        img1, _ = _render(sc, cam, 1, False)
        flips = np.abs(img - img1) > 2e-4   # (a cut or stop decided the other way)
        assert flips.mean() < 1e-3
