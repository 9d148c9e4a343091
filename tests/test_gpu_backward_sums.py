"""The backward kernels' sums over pixels as matrix products: lists around the 8-row blocks and
256-entry chunks against the FP64 oracle (the bars of test_gpu_backward / test_gpu_backward_mfma),
every row in every quadrant against the quadrant lists, and an upstream gradient that is not
finite, which may reach only the Gaussians its pixel blends."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note
from test_gpu_backward import FIELDS, _case, _compare
from test_gpu_backward_mfma import SPLITS, _compare as _compare_mfma, _forward_state

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    """n faint Gaussians over one or few tiles, so that no pixel stops early and lists stay long."""
    sc = scenes.camera_box_scene(n, seed=seed, log_scale_mu=float(np.log(0.5)))
    sc.opacity[:] = 0.004 + 0.02 * sc.opacity
    return sc


def _backward(proj, bins, cam, dimg, bg, n, prec, all_rows=False):
    import torch
    grads = gs.Grads(n)
    d = torch.from_numpy(np.ascontiguousarray(dimg, np.float32)).cuda()
    opt = gs.options(precision=prec, splits=SPLITS.get(prec, 2), bg=bg, all_rows=all_rows)
    if prec == "fp32":
        gs.gs_rasterize_backward(proj, bins, cam, opt, d, grads)
    else:
        _, aux = _forward_state(proj, bins, cam, opt)
        gs.gs_rasterize_backward_mfma(proj, bins, cam, opt, d, aux[0], aux[1], grads)
    torch.cuda.synchronize()
    return {f: getattr(grads, f).cpu().numpy().astype(np.float64)[:n] for f in FIELDS}


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("n,w,h", [(1, 16, 16), (7, 16, 16), (8, 9, 7), (9, 17, 16), (255, 16, 16), (256, 16, 16),
                                   (257, 16, 16), (513, 16, 16), (600, 40, 23)])
def test_list_lengths(n, w, h, prec):
    note(f"backward sums {prec}: n {n}, {w}x{h}")
    sc, cam, bg = _scene(n, 100 + n), scenes.pinhole(w, h, 60.0), (0.2, 0.1, 0.3)
    _, _, _, dimg, _, ref, proj, bins = _case(sc, cam, bg, 5)
    cmp = _compare if prec == "fp32" else _compare_mfma
    got = _backward(proj, bins, cam, dimg, bg, n, prec)
    cmp(f"{prec} n={n}", got, ref)
    # the same sums with every row in every quadrant: FP32 sums in another order only
    full = _backward(proj, bins, cam, dimg, bg, n, prec, all_rows=True)
    for f in FIELDS:
        assert np.abs(full[f] - got[f]).max() <= 2e-5 * max(np.abs(got[f]).max(), 1e-30), f


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_upstream_stays_with_its_pixel(prec, value):
    note(f"backward sums {prec}: upstream {value}")
    n, bg = 300, (0.0, 0.0, 0.0)
    sc, cam = scenes.camera_box_scene(n, seed=9, log_scale_mu=float(np.log(0.08))), scenes.pinhole(40, 32, 60.0)
    _, _, _, dimg, _, _, proj, bins = _case(sc, cam, bg, 6)
    y, x = 13, 21
    only = np.zeros_like(dimg)
    only[:, y, x] = 1.0
    hit = np.abs(_backward(proj, bins, cam, only, bg, n, prec)["rgb"]).max(1) > 0   # blended by the pixel
    assert 0 < hit.sum() < n
    dimg[:, y, x] = 0.0
    want = _backward(proj, bins, cam, dimg, bg, n, prec)
    dimg[1, y, x] = value
    got = _backward(proj, bins, cam, dimg, bg, n, prec)
    for f in FIELDS:
        a, b = got[f].reshape(n, -1), want[f].reshape(n, -1)
        assert np.isfinite(a[~hit]).all(), f
        assert np.abs(a - b)[~hit].max() <= 2e-5 * np.abs(b).max(), f
    assert not np.isfinite(got["rgb"][hit][:, 1]).any()   # (alpha T times the value)
    assert np.isfinite(got["rgb"][:, [0, 2]]).all()
