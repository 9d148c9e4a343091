"""The FP32 quadrant lists on long thin splats across a large frame, where the FP32 power itself is off
by more than a fixed margin of the quadrant test (its terms reach 1e7 and cancel): the image and
every auxiliary plane bit-identical to the rasterizer that runs every row in every quadrant, and
the backward pass blending the same pairs.

Colour gradients under an upstream gradient of one are sums of positive terms alpha T: a
quadrant left out takes its share away, and the sums differ otherwise only by the order of one FP32
addition per tile of at most 4,000, 4,000 x 2^-24 = 2.4e-4 if all rounded the same way (one
quadrant in a thousand is 1e-3)."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note
from test_gpu_fp32_lists import AUX

pytestmark = pytest.mark.gpu

N = 48


def _scene(width, sigma_px, seed):
    """Splats at depth 4 around the view's axis, turned in the image plane, `sigma_px` long and thin
    down to the projection's floor; half of them so faint that every blended pair lies at the cut."""
    rng = np.random.default_rng(seed)
    sc = scenes.camera_box_scene(N, seed=seed)
    cam = scenes.pinhole(width, width * 9 // 16, 60.0)
    sc.mean[0] = rng.uniform(-1.5, 1.5, N)
    sc.mean[1] = rng.uniform(-0.8, 0.8, N)
    sc.mean[2] = 4.0
    sc.log_scale[:] = -12.0
    sc.log_scale[0] = np.log(sigma_px * 4.0 / cam.fx) + rng.uniform(-0.5, 0.5, N)
    ang = rng.uniform(0, np.pi, N)
    sc.quat[:] = 0.0
    sc.quat[0], sc.quat[3] = np.cos(ang / 2), np.sin(ang / 2)
    sc.opacity[:] = np.where(np.arange(N) % 2 == 0, rng.uniform(1.002, 1.05, N) / 255, rng.uniform(0.02, 0.5, N))
    return sc, cam


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("width,sigma_px", [(1920, 600.0), (7680, 2500.0)])
def test_forward_is_that_of_every_row(width, sigma_px, group):
    import torch
    note(f"fp32 long splats: {width} wide, sigma {sigma_px}, group {group}")
    sc, cam = _scene(width, sigma_px, 5)
    ds = gs.DeviceScene(sc)
    out = []
    for all_rows in (False, True):
        r = gs.Renderer(sc.n, cam.width, cam.height, group=group)
        r.render(ds, cam, gs.options(group=group, precision="fp32", aux_flags=AUX, all_rows=all_rows))
        torch.cuda.synchronize()
        out.append((r.image, r.aux))
    assert float(out[1][1][1].max()) > 0.01    # something is blended
    for a, b in zip(*out):
        assert torch.equal(a, b), int((a != b).sum())


@pytest.mark.parametrize("width,sigma_px", [(1920, 600.0), (7680, 2500.0)])
def test_backward_blends_the_same_pairs(width, sigma_px):
    import torch
    note(f"fp32 long splats backward: {width} wide, sigma {sigma_px}")
    sc, cam = _scene(width, sigma_px, 6)
    ds = gs.DeviceScene(sc)
    r = gs.Renderer(sc.n, cam.width, cam.height)
    r.render(ds, cam, gs.options(precision="fp32"))
    up = torch.ones((3, cam.height, cam.width), dtype=torch.float32, device="cuda")
    got = []
    for all_rows in (False, True):
        grads = gs.Grads(sc.n)
        gs.gs_rasterize_backward(r.proj, r.bins, cam, gs.options(precision="fp32", all_rows=all_rows), up, grads)
        torch.cuda.synchronize()
        got.append(grads.rgb.cpu().numpy().astype(np.float64))
    assert (got[1].sum(1) > 0).sum() > N // 2
    rel = np.abs(got[0] - got[1]) / np.maximum(got[1], 1e-30)
    print(f"{width} wide: colour gradients differ by at most {rel.max():.2e}")
    assert rel.max() <= 2.4e-4
