"""The depth sort around its tiles, groups of tiles and rows of counts: the visible Gaussians' order
equal to a stable sort of their depth bits, for lists of one tile up to more than the row
scheme takes, with depths of few and of many octaves and many equal ones."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu


# one workgroup up to 8,192 Gaussians; 1,024-key tiles up to 2^20 Gaussians, in groups of 4 (a wave's rows: 64 tiles ungrouped, 256 grouped);
# 2,048-key tiles above, in rows up to 2^21
@pytest.mark.parametrize("n", [2, 65, 1023, 1025, 4097, 8192, 8193, 66000, 270000, (1 << 20) + 1, (1 << 21) + 1])
def test_depth_order_is_a_stable_sort(n):
    import torch
    note(f"depth order: n {n}")
    sc = scenes.camera_box_scene(n, seed=3, log_scale_mu=float(np.log(0.002)))
    rng = np.random.default_rng(n)
    z = np.exp(rng.uniform(np.log(0.5), np.log(5000.0), n)).astype(np.float32)
    z[: n // 4] = rng.choice(np.array([0.5, 1.0, 1.5, 3.0], np.float32), n // 4)
    z[n // 4: n // 2] = np.float32(2.0) + rng.integers(0, 3, n // 2 - n // 4).astype(np.float32) * 2.0 ** -20
    sc.mean[0] = sc.mean[1] = 0.0
    sc.mean[2] = z
    cam = scenes.pinhole(64, 48, 60.0)
    r = gs.Renderer(n, cam.width, cam.height, group=1)
    ds = gs.DeviceScene(sc)
    for dev in (False, True):
        r.render(ds, cam, gs.options(precision="fp16", device_counts=dev))
        torch.cuda.synchronize()
        count = r.proj.count.cpu().numpy().view(np.uint32)
        depth = r.proj.rgb.cpu().numpy().view(np.uint32)[:, 3]
        seen = np.nonzero(count)[0]
        assert seen.size == n
        want = seen[np.argsort(depth[seen], kind="stable")]
        assert np.array_equal(r.proj.order.cpu().numpy().view(np.uint32)[:n], want)
