"""Gradients of splats down to the 0.3 px^2 floor of the projected variance, at tile corners, edges and
centres, each Gaussian held to its own size: the offsets from the centre are a fraction of a
pixel there, so sums over pixels that are taken about another point and shifted cancel.

One splat per 32x32 pixels and nothing else near it; centres are multiples of 1/64 pixel, so every
offset is exact in FP32.

One pixel with an upstream gradient per splat: all sums hold that pixel's p alone, so the conic and
centre gradients are fixed multiples of the opacity gradient, whatever alpha's own rounding is.  p dx dx
rounds twice, (a dx + b dy) p up to four times, and p = o dL/do within 2.5 ulp of a division and one of
the read-back: under 7 units of 2^-24 in all, the bar is 12.

Every pixel, against the FP64 oracle: error over the sum of the terms' sizes.  D = log2(alpha_raw) has
three coefficients within 2 units of 2^-24, four roundings and a logarithm, on terms of at most
16 together (log2 255 for the alphas that count, twice over for the mixed term of |b| <= sqrt(ac) / 2): 6
units of 16, times ln 2 = 4e-6 of alpha; the step to p and the sums of at most 64 x 4 terms, 1e-6
each: 6e-6."""
import numpy as np
import pytest

from oracle import oracle
from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note
from test_gpu_backward import FIELDS, _gpu_backward, _upload
from test_gpu_backward_mfma import _gpu_backward_mfma

pytestmark = pytest.mark.gpu

CELLS = 16    # splats a side
ULP = 2.0 ** -24


def _splats(variance, seed):
    """Records and tile lists: splat (i, j) near the tile corner at 32 (i, j) + 16, offset by up to a
    tile to each side and often by a whole or half tile, where the centre is on an edge or at a tile's middle."""
    rng = np.random.default_rng(seed)
    n = CELLS * CELLS
    off = rng.integers(-512, 513, size=(n, 2)) / 64.0
    near = rng.random((n, 2)) < 0.6                     # within half a pixel of the corner or the middle
    off[near] = rng.choice([0.0, 8.0, -8.0], size=near.sum()) + rng.integers(-31, 32, size=near.sum()) / 64.0
    cell = np.stack(np.meshgrid(np.arange(CELLS), np.arange(CELLS)), -1).reshape(-1, 2)
    xy = 32.0 * cell + 16.0 + off
    vx, vy = variance * np.exp(rng.uniform(0, 0.5, (2, n)))
    vxy = rng.uniform(-0.5, 0.5, n) * np.sqrt(vx * vy)
    det = vx * vy - vxy * vxy
    conic = np.stack([vy / det, -vxy / det, vx / det], 1).astype(np.float32).astype(np.float64)
    opacity = rng.uniform(0.5, 0.95, n).astype(np.float32).astype(np.float64)
    rgb = rng.uniform(0.2, 1.0, (n, 3)).astype(np.float32).astype(np.float64)
    rec = dict(xy=xy, conic=conic, opacity=opacity, rgb=rgb, depth=np.full(n, 2.0),
               flags=np.zeros(n, np.uint32))
    cam = scenes.pinhole(32 * CELLS, 32 * CELLS, 60.0)
    tx = cam.width // 16
    r = 3.4 * np.sqrt(np.maximum(vx, vy))               # alpha < 1/255 beyond
    lists = [[] for _ in range(tx * tx)]
    for g in range(n):
        x0, y0 = np.floor((xy[g] - r[g]) / 16).astype(int)
        x1, y1 = np.floor((xy[g] + r[g]) / 16).astype(int)
        for y in range(max(y0, 0), min(y1, tx - 1) + 1):
            for x in range(max(x0, 0), min(x1, tx - 1) + 1):
                lists[y * tx + x].append(g)
    start = np.cumsum([0] + [len(v) for v in lists])
    return rec, start, np.array([g for v in lists for g in v], np.int64), cam


def _backward(prec, rec, start, ids, cam, dimg):
    proj, bins = _upload(rec, start, ids)
    n, bg = rec["depth"].size, (0.0, 0.0, 0.0)
    if prec == "fp32":
        return _gpu_backward(proj, bins, cam, dimg, bg, n)
    return _gpu_backward_mfma(proj, bins, cam, dimg, bg, n, prec)


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("variance", [0.3, 1.0, 10.0])
def test_one_pixel(variance, prec):
    note(f"backward small splats, one pixel: {prec}, variance {variance}")
    rec, start, ids, cam = _splats(variance, 11)
    n = rec["depth"].size
    pix = np.floor(rec["xy"]).astype(int)
    dimg = np.zeros((3, cam.height, cam.width))
    dimg[:, pix[:, 1], pix[:, 0]] = np.random.default_rng(12).normal(size=(3, n))
    got = _backward(prec, rec, start, ids, cam, dimg)
    p = got["opacity"] * rec["opacity"]
    assert (p != 0).all()
    dx, dy = (pix + 0.5 - rec["xy"]).T
    a, b, c = rec["conic"].T
    want = {"conic": np.stack([-0.5 * dx * dx, -dx * dy, -0.5 * dy * dy], 1) * p[:, None],
            "xy": np.stack([a * dx + b * dy, b * dx + c * dy], 1) * p[:, None]}
    size = {"conic": np.abs(want["conic"]),
            "xy": np.stack([np.abs(a * dx) + np.abs(b * dy), np.abs(b * dx) + np.abs(c * dy)], 1) * np.abs(p)[:, None]}
    for f in want:
        rel = np.abs(got[f] - want[f]) / np.maximum(size[f], 1e-30)
        print(f"{prec} variance {variance} {f}: max {rel.max():.2e} of the term")
        assert rel.max() <= 12 * ULP, (f, int(rel.max(1).argmax()))


@pytest.mark.parametrize("variance", [0.3, 1.0, 10.0])
def test_every_pixel(variance):
    note(f"backward small splats, every pixel: variance {variance}")
    rec, start, ids, cam = _splats(variance, 13)
    dimg = np.random.default_rng(14).normal(size=(3, cam.height, cam.width))
    dimg[:, oracle.composite(rec, cam, start, ids)["ambiguous"] != 0] = 0.0
    dimg = dimg.astype(np.float32).astype(np.float64)
    got = _backward("fp32", rec, start, ids, cam, dimg)
    ref = oracle.composite_backward(rec, cam, start, ids, dimg)
    pos = oracle.composite_backward(rec, cam, start, ids, np.abs(dimg))   # (one splat deep: every p >= 0)
    a, b, c = np.abs(rec["conic"]).T
    m0 = pos["opacity"] * rec["opacity"]
    sxx, syy = -2 * pos["conic"][:, 0], -2 * pos["conic"][:, 2]
    size = {"rgb": pos["rgb"], "opacity": pos["opacity"],
            "conic": np.stack([sxx / 2, np.sqrt(sxx * syy), syy / 2], 1),
            "xy": np.stack([a * np.sqrt(sxx * m0) + b * np.sqrt(syy * m0), b * np.sqrt(sxx * m0) + c * np.sqrt(syy * m0)], 1)}
    for f in FIELDS:
        rel = np.abs(got[f] - ref[f]) / size[f]
        print(f"variance {variance} {f}: mean {rel.mean():.2e}, max {rel.max():.2e} of the terms")
        assert rel.max() <= 6e-6, f
