"""Measured workloads of the renderer: frames, serving stages and training steps.

Each case is one call that a program using the library makes in earnest, through
`gs.Renderer`, the stage functions and the backward passes:

  frame   a scene on the device to an image on the device (`gs.Renderer.render`)
  prep    the preparation half of a served request (`gs.gs_preprocess`, `gs.gs_bin_sort`)
  batch   the raster half of several served requests in one launch (`gs.gs_rasterize_batch`)
  train   a frame, then the gradients of its compositing (`gs.gs_rasterize_backward` for FP32,
          `gs.gs_rasterize_backward_mfma` from the forward's state for FP16/BF16)

Scenes follow the synthetic workloads of `paper_2605_17855_amd/scenes.py` (camera-space box,
clustered world-space scene, dense overlap stress), drawn here on the GPU from the seed alone;
the camera of a world-space scene is a random pose on the radius-4 sphere.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_2605_17855_amd import gs

TILE = 16


def _case(name, kind, scene, n, width, height, precision, group=1, splits=2, tight=False, sh=3, bg=0.0, jobs=1):
    return {"name": name, "kind": kind, "scene": scene, "n": n, "width": width, "height": height,
            "precision": precision, "group": group, "splits": splits, "tight": tight, "sh": sh, "bg": bg,
            "jobs": jobs}


def listed():
    return [
        # the smallest call: a thumbnail of a small model, where launches and latency are all there is
        _case("frame_4k_128_fp32", "frame", "box", 4096, 128, 128, "fp32", sh=0),
        # the smallest served request: the smallest scene and resolution of the serving mix, with its
        # options (FP16, opacity-aware culling)
        _case("frame_500k_360p_fp16_tight", "frame", "clustered", 500_000, 640, 360, "fp16", tight=True),
        # the ordinary frame: 1M Gaussians at 1080p, tensorized and plain
        _case("frame_1m_1080p_fp16", "frame", "clustered", 1_000_000, 1920, 1080, "fp16"),
        _case("frame_1m_1080p_fp32", "frame", "clustered", 1_000_000, 1920, 1080, "fp32"),
        # the same frame with the tighter tile lists
        _case("frame_1m_1080p_fp16_tight", "frame", "clustered", 1_000_000, 1920, 1080, "fp16", tight=True),
        # a large scene with 2x2 tile groups in BF16 (three pieces per coefficient)
        _case("frame_3m_1080p_bf16_g2", "frame", "clustered", 3_000_000, 1920, 1080, "bf16", group=2, splits=3),
        # the same scene size at 4K, ungrouped: the most pixels and sorted entries of an ordinary scene
        _case("frame_3m_2160p_fp16", "frame", "clustered", 3_000_000, 3840, 2160, "fp16"),
        # the dense stress scene with 4x4 groups: the most Gaussians and overlap
        _case("frame_6m_dense_1080p_fp16_g4", "frame", "dense", 6_000_000, 1920, 1080, "fp16", group=4),
        # a served request's preparation at the largest served resolution
        _case("prep_2m_1440p_tight", "prep", "clustered", 2_000_000, 2560, 1440, "fp16", tight=True),
        # the raster launch of four served requests at once (one of each served resolution)
        _case("batch_4_fp16_tight", "batch", "clustered", 1_000_000, 2560, 1440, "fp16", tight=True, jobs=4),
        # training steps: the plain FP32 path at 1080p, and the tensorized one at an odd size of the
        # paper's workloads with a background
        _case("train_1m_1080p_fp32", "train", "clustered", 1_000_000, 1920, 1080, "fp32"),
        _case("train_300k_979x546_fp16", "train", "clustered", 300_000, 979, 546, "fp16", bg=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "prep", "batch", "train"])
    scene = "clustered"
    if kind == "frame":
        scene = rng.choice(["box", "clustered", "clustered", "clustered", "dense"])
    n = {"box": _log_int(rng, 1024, 65536), "dense": _log_int(rng, 200_000, 4_000_000),
         "clustered": _log_int(rng, 20_000, 1_000_000 if kind in ("train", "batch") else 2_000_000)}[scene]
    width = _log_int(rng, 128, 512) if scene == "box" else _log_int(rng, 320, 1920 if kind == "train" else 2560)
    height = max(64, int(width * rng.uniform(0.5, 0.75)))
    precision = rng.choice(["fp32", "fp16", "fp16", "bf16"])
    group = 1
    if kind == "frame" and precision != "fp32":
        group = rng.choice([4, 8] if scene == "dense" else [1, 1, 2, 4, 8])
    elif scene == "dense":
        group = 4
    c = _case("", kind, scene, n, width, height, precision, group=group,
              splits=3 if precision == "bf16" else 2,
              tight=kind in ("prep", "batch") or (kind == "frame" and rng.random() < 0.3),
              sh=0 if scene == "box" else rng.choice([1, 2, 3, 3]), bg=rng.choice([0.0, 0.5]),
              jobs=rng.randint(2, 6) if kind == "batch" else 1)
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------------------

def _scene_arrays(case, seed):
    """mean (3, n), log_scale (3, n), quat (4, n), opacity (n), sh (n, (deg+1)^2 * 3), FP32 on the GPU."""
    n, deg = case["n"], case["sh"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    nb = (deg + 1) ** 2

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    def uniform(*shape):
        return torch.rand(shape, generator=gen, device="cuda")

    if case["scene"] == "box":
        mean = torch.stack([uniform(n) * 2 - 1, uniform(n) * 2 - 1, uniform(n) * 4 + 2])
        ls_mu, ls_sigma, op_mu, op_sigma = math.log(0.02), 0.5, 0.0, 1.0
    else:
        clusters = 256 if n >= 2_500_000 and case["scene"] == "clustered" else 64
        centres = uniform(clusters, 3) * 10 - 5
        sigma = 0.25 + 0.75 * uniform(clusters)
        comp = torch.randint(0, clusters, (n,), generator=gen, device="cuda")
        mean = (centres[comp].T + sigma[comp][None, :] * normal(3, n)).clamp_(-5, 5)
        ls_mu, ls_sigma, op_mu, op_sigma = math.log(0.01), 0.7, 0.0, 1.5
        if case["scene"] == "dense":
            ls_mu, ls_sigma, op_mu, op_sigma = math.log(0.05), 0.5, -1.0, 1.0
    quat = normal(4, n)
    sh = normal(n, nb * 3).mul_(0.2)
    sh[:, :3] = uniform(n, 3) - (0.5 if case["scene"] == "box" else 0.0)
    if case["scene"] == "box":
        sh[:, :3] /= 0.5 / math.sqrt(math.pi)
    return (mean.contiguous(), normal(3, n).mul_(ls_sigma).add_(ls_mu), (quat / quat.norm(dim=0)).contiguous(),
            torch.sigmoid(normal(n) * op_sigma + op_mu), sh)


def _camera(case, seed, width, height):
    """Square-pixel pinhole of 60 degrees, at the origin for the camera-space box, else looking at
    the origin from a random point of the radius-4 sphere (x right, y down, z forward)."""
    R, t = np.eye(3), np.zeros(3)
    if case["scene"] != "box":
        rng = np.random.default_rng(seed)
        z, phi = rng.uniform(-0.9, 0.9), rng.uniform(0, 2 * math.pi)
        s = math.sqrt(1 - z * z)
        p = 4.0 * np.array([s * math.cos(phi), s * math.sin(phi), z])
        f = -p / np.linalg.norm(p)
        r = np.cross(f, [0.0, 0.0, 1.0])
        r /= np.linalg.norm(r)
        R = np.stack([r, np.cross(f, r), f])
        t = -(R.astype(np.float32).astype(np.float64) @ p)
    fx = float(np.float32(width / 2 / math.tan(math.radians(30))))
    return types.SimpleNamespace(R=R.astype(np.float32), t=t.astype(np.float32), fx=fx, fy=fx, cx=width / 2,
                                 cy=height / 2, width=width, height=height, znear=float(np.float32(0.2)))


def _cameras(case, seed):
    """One camera; a batch takes further poses at the served resolutions' share of its own."""
    share = (1.0, 0.75, 0.5, 0.25)
    w, h = case["width"], case["height"]
    return [_camera(case, seed + 7919 * j, max(16, int(w * share[j % 4])), max(16, int(h * share[j % 4])))
            for j in range(case["jobs"])]


class _DeviceScene:
    """Scene tensors that are on the GPU already, as the library takes them."""

    def __init__(self, case, seed):
        self.arrays = _scene_arrays(case, seed)
        self.n, self.sh_degree = case["n"], case["sh"]
        s = gs.gs_scene()
        s.n, s.sh_degree = self.n, self.sh_degree
        s.mean, s.log_scale, s.quat, s.opacity, s.sh = (a.data_ptr() for a in self.arrays)
        self.struct = s


def _options(case):
    aux = gs.GS_AUX_TFINAL | gs.GS_AUX_LAST if case["kind"] == "train" and case["precision"] != "fp32" else 0
    return gs.options(group=case["group"], precision=case["precision"], splits=case["splits"],
                      bg=(case["bg"],) * 3, tight=case["tight"], aux_flags=aux)


def prepare(case, seed):
    s = types.SimpleNamespace(kind=case["kind"], precision=case["precision"], opt=_options(case))
    s.scene = _DeviceScene(case, seed)
    s.cams = _cameras(case, seed)
    s.renderers = []
    for cam in s.cams:
        r = gs.Renderer(case["n"], cam.width, cam.height, group=case["group"],
                        capacity=8 * case["n"] if s.kind == "prep" else 0)
        r.render(s.scene, cam, s.opt)   # the entry buffers grow to the scene as on a program's first frame
        if s.kind == "prep":            # the whole entry buffers come back: nothing stale past the entries
            r.bins.keys.zero_()
            r.bins.vals.zero_()
        s.renderers.append(r)
    if s.kind == "batch":
        s.counter = torch.zeros(gs.BATCH_COUNTER_WORDS, dtype=torch.int32, device="cuda")
        s.items = [(r.proj, r.bins, cam, r.image, None) for r, cam in zip(s.renderers, s.cams)]
    if s.kind == "train":
        gen = torch.Generator(device="cuda").manual_seed(seed + 1)
        s.dimage = torch.randn((3, case["height"], case["width"]), generator=gen, device="cuda")
        s.grads = gs.Grads(case["n"])
    return s


def run(s):
    ren, cam = s.renderers[0], s.cams[0]
    if s.kind == "frame":
        n_keys = ren.render(s.scene, cam, s.opt)
        return {"image": ren.image, "n_keys": n_keys}
    if s.kind == "prep":
        gs.gs_preprocess(s.scene, cam, s.opt, ren.proj, ren.ws)
        n_keys = gs.gs_bin_sort(ren.proj, cam, s.opt, ren.bins, ren.ws)
        return {"n_keys": n_keys, "keys": ren.bins.keys, "vals": ren.bins.vals, "ranges": ren.bins.ranges}
    if s.kind == "batch":
        gs.gs_rasterize_batch(s.items, s.opt, s.counter)
        return {"images": [r.image for r in s.renderers]}
    ren.render(s.scene, cam, s.opt)
    s.grads.zero_()
    out = {"image": ren.image}
    if s.precision == "fp32":
        gs.gs_rasterize_backward(ren.proj, ren.bins, cam, s.opt, s.dimage, s.grads)
    else:
        gs.gs_rasterize_backward_mfma(ren.proj, ren.bins, cam, s.opt, s.dimage, ren.aux[0], ren.aux[1], s.grads)
        out["t_final"] = ren.aux[0]
    g = s.grads
    out.update(rgb=g.rgb, opacity=g.opacity, conic=g.conic, xy=g.xy)
    return out


# Gaussians blended per pixel before its stop, roughly, by scene (the orbit views of the 1M
# clustered scene blend 36)
_BLENDS = {"box": 10, "clustered": 36, "dense": 60}


def work(case):
    n, nb = case["n"], (case["sh"] + 1) ** 2
    scene = n * (44 + 12 * nb)                       # every scene array read once
    cams = [(max(16, int(case["width"] * f)), max(16, int(case["height"] * f)))
            for f in ((1.0, 0.75, 0.5, 0.25)[j % 4] for j in range(case["jobs"]))]
    pixels = sum(w * h for w, h in cams)
    pairs = pixels * _BLENDS[case["scene"]]
    flops = 23 * pairs                               # power, alpha and blend of each blended pair
    image = 12 * pixels
    if case["kind"] == "prep":
        # scene in; a key and an index per (visible Gaussian, tile), at least one per visible Gaussian
        return {"bytes": scene + 12 * n // 5 + 8 * pixels // 256, "flops": 200 * n}
    if case["kind"] == "batch":
        return {"bytes": image + 4 * pixels // 256 * 100 + 40 * n // 5 * case["jobs"], "flops": flops}
    if case["kind"] == "train":
        return {"bytes": scene + 2 * image + 36 * n, "flops": 3 * flops + 200 * n}
    return {"bytes": scene + image, "flops": flops + 200 * n}


# ---- 64-bit values ------------------------------------------------------------------------

def _project64(arrays, deg, cam):
    """Screen-space records of the visible Gaussians in (depth, index) order, in FP64."""
    mean, log_scale, quat, opacity, sh = arrays
    d = torch.float64
    R = torch.tensor(cam.R, dtype=d, device="cuda")
    t = torch.tensor(cam.t, dtype=d, device="cuda")
    p = R @ mean.to(d) + t[:, None]
    keep = torch.nonzero(p[2] > cam.znear).flatten()
    p = p[:, keep]
    z = p[2]
    q = quat[:, keep].to(d)
    w, x, y, k = q / q.norm(dim=0)
    M = torch.stack([torch.stack([1 - 2 * (y * y + k * k), 2 * (x * y - w * k), 2 * (x * k + w * y)]),
                     torch.stack([2 * (x * y + w * k), 1 - 2 * (x * x + k * k), 2 * (y * k - w * x)]),
                     torch.stack([2 * (x * k - w * y), 2 * (y * k + w * x), 1 - 2 * (x * x + y * y)])])
    MS = M * torch.exp(log_scale[:, keep].to(d))[None]
    ux = (p[0] / z).clamp(-1.3 * cam.width / 2 / cam.fx, 1.3 * cam.width / 2 / cam.fx)
    uy = (p[1] / z).clamp(-1.3 * cam.height / 2 / cam.fy, 1.3 * cam.height / 2 / cam.fy)
    T0 = (cam.fx / z) * (R[0][:, None] - ux * R[2][:, None])
    T1 = (cam.fy / z) * (R[1][:, None] - uy * R[2][:, None])
    P0, P1 = (T0[:, None] * MS).sum(0), (T1[:, None] * MS).sum(0)
    sxx, syy, sxy = (P0 * P0).sum(0) + 0.3, (P1 * P1).sum(0) + 0.3, (P0 * P1).sum(0)
    c = torch.linalg.cross(P0, P1, dim=0)
    det = (c * c).sum(0) + 0.3 * (sxx + syy - 0.6) + 0.09
    mx, my = cam.fx * p[0] / z + cam.cx, cam.fy * p[1] / z + cam.cy
    r = 3 * torch.sqrt((sxx + syy) / 2 + torch.sqrt(((sxx - syy) / 2) ** 2 + sxy * sxy))
    TX, TY = -(-cam.width // TILE), -(-cam.height // TILE)
    x0, x1 = torch.floor((mx - r) / TILE).clamp(min=0), torch.floor((mx + r) / TILE).clamp(max=TX - 1)
    y0, y1 = torch.floor((my - r) / TILE).clamp(min=0), torch.floor((my + r) / TILE).clamp(max=TY - 1)
    vis = torch.nonzero((x0 <= x1) & (y0 <= y1)).flatten()
    vis = vis[torch.sort(z[vis].float(), stable=True).indices]
    ids = keep[vis]
    centre = -(R.T @ t)
    v = mean[:, ids].to(d) - centre[:, None]
    bx, by, bz = v / v.norm(dim=0)
    basis = [torch.full_like(bx, 0.5 / math.sqrt(math.pi))]
    if deg >= 1:
        a = math.sqrt(3 / (4 * math.pi))
        basis += [-a * by, a * bz, -a * bx]
    if deg >= 2:
        a, b = math.sqrt(15 / (4 * math.pi)), math.sqrt(5 / (16 * math.pi))
        basis += [a * bx * by, -a * by * bz, b * (3 * bz * bz - 1), -a * bx * bz, a / 2 * (bx * bx - by * by)]
    if deg >= 3:
        a, b = math.sqrt(35 / (32 * math.pi)), math.sqrt(105 / (4 * math.pi))
        e, f = math.sqrt(21 / (32 * math.pi)), math.sqrt(7 / (16 * math.pi))
        basis += [-a * by * (3 * bx * bx - by * by), b * bx * by * bz, -e * by * (5 * bz * bz - 1),
                  f * bz * (5 * bz * bz - 3), -e * bx * (5 * bz * bz - 1), b / 2 * bz * (bx * bx - by * by),
                  -a * bx * (bx * bx - 3 * by * by)]
    coef = sh[ids].to(d).view(len(ids), -1, 3)
    rgb = ((coef * torch.stack(basis, 1)[:, :, None]).sum(1) + 0.5).clamp(min=0)
    rec = torch.stack([mx[vis], my[vis], (syy / det)[vis], (-sxy / det)[vis], (sxx / det)[vis],
                       opacity[ids].to(d), rgb[:, 0], rgb[:, 1], rgb[:, 2]], 1)
    rect = torch.stack([x0[vis], y0[vis], x1[vis], y1[vis]], 1).long()
    return rec, rect, ids, TX, TY


def _tile_lists(rect, TX, TY):
    wd, ht = rect[:, 2] - rect[:, 0] + 1, rect[:, 3] - rect[:, 1] + 1
    cnt = wd * ht
    first = torch.cumsum(cnt, 0) - cnt
    g = torch.repeat_interleave(torch.arange(len(cnt), device="cuda"), cnt)
    j = torch.arange(len(g), device="cuda") - first[g]
    tile = ((rect[g, 1] + j // wd[g]) * TX + rect[g, 0] + j % wd[g]).int()
    del j
    tile, order = torch.sort(tile, stable=True)
    g = g[order]
    num = torch.bincount(tile, minlength=TX * TY)
    return g, torch.cumsum(num, 0) - num, num


def _walk(rec, lists, cam, TX, TY, visit):
    """Front to back through every tile's list, one list position at a time over the tiles that
    still blend: visit(tiles, record row, dx, dy, alpha, T before, blended here).  Returns the final T."""
    g, start, num = lists
    d = torch.float64
    px = torch.arange(TILE * TILE, device="cuda")
    ix, iy = px % TILE, px // TILE
    T_all = torch.ones((TX * TY, TILE * TILE), dtype=d, device="cuda")
    at = torch.nonzero(num > 0).flatten()
    j, T, alive = 0, None, None
    while True:
        if j % 32 == 0:
            if T is not None:
                T_all[at] = T
                on = torch.nonzero((num[at] > j) & alive.any(1)).flatten()
                at, alive = at[on], alive[on]
            if not len(at):
                return T_all
            X, Y = (at % TX)[:, None] * TILE + ix, (at // TX)[:, None] * TILE + iy
            T = T_all[at]
            if alive is None:
                alive = (X < cam.width) & (Y < cam.height)
        here = (num[at] > j)[:, None]
        row = g[(start[at] + j).clamp(max=len(g) - 1)]
        r = rec[row]
        dx, dy = X + 0.5 - r[:, 0:1], Y + 0.5 - r[:, 1:2]
        power = -0.5 * (r[:, 2:3] * dx * dx + r[:, 4:5] * dy * dy) - r[:, 3:4] * dx * dy
        raw = r[:, 5:6] * torch.exp(power)
        alpha = raw.clamp(max=0.99)
        on = alive & here & (raw >= 1 / 255)
        Tn = T * (1 - alpha)
        stop = on & (Tn < 1e-4)
        alive = alive & ~stop
        on = on & ~stop
        visit(at, row, r, dx, dy, raw, alpha, T, on)
        T = torch.where(on, Tn, T)
        j += 1


def _image64(case, rec, lists, cam, TX, TY):
    C = torch.zeros((3, TX * TY, TILE * TILE), dtype=torch.float64, device="cuda")

    def blend(at, row, r, dx, dy, raw, alpha, T, on):
        wgt = torch.where(on, alpha * T, torch.zeros_like(T))
        for c in range(3):
            C[c].index_add_(0, at, wgt * r[:, 6 + c:7 + c])

    T = _walk(rec, lists, cam, TX, TY, blend)
    return C, T


def _plane(tiles, cam, TX, TY):
    """(tiles, 256) to (H, W)."""
    p = tiles.view(TY, TX, TILE, TILE).permute(0, 2, 1, 3).reshape(TY * TILE, TX * TILE)
    return p[:cam.height, :cam.width].contiguous()


def _tiles(plane, TX, TY):
    out = torch.zeros((TY * TILE, TX * TILE), dtype=torch.float64, device="cuda")
    out[:plane.shape[0], :plane.shape[1]] = plane
    return out.view(TY, TILE, TX, TILE).permute(0, 2, 1, 3).reshape(TY * TX, TILE * TILE)


def exact(case, seed):
    if case["kind"] == "prep":
        return None   # whole numbers only
    arrays = _scene_arrays(case, seed)
    images = []
    for cam in _cameras(case, seed):
        rec, rect, ids, TX, TY = _project64(arrays, case["sh"], cam)
        lists = _tile_lists(rect, TX, TY)
        C, T = _image64(case, rec, lists, cam, TX, TY)
        images.append(torch.stack([_plane(C[c] + T * case["bg"], cam, TX, TY) for c in range(3)]))
    if case["kind"] == "frame":
        return {"image": images[0], "n_keys": None}
    if case["kind"] == "batch":
        return {"images": images}

    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    dimage = torch.randn((3, case["height"], case["width"]), generator=gen, device="cuda")
    dl = torch.stack([_tiles(dimage[c], TX, TY) for c in range(3)])
    grad = torch.zeros((len(rec), 9), dtype=torch.float64, device="cuda")
    left = torch.stack([C[c] + T * case["bg"] for c in range(3)])   # colour behind the position reached

    def gradients(at, row, r, dx, dy, raw, alpha, Tb, on):
        wgt = torch.where(on, alpha * Tb, torch.zeros_like(Tb))
        dalpha = torch.zeros_like(Tb)
        terms = []
        for c in range(3):
            col = r[:, 6 + c:7 + c]
            left[c].index_add_(0, at, -wgt * col)
            g = dl[c][at]
            dalpha += g * (col * Tb - left[c][at] / (1 - alpha))
            terms.append((wgt * g).sum(1))
        dp = torch.where(on & (raw < 0.99), dalpha * alpha, torch.zeros_like(Tb))
        terms += [dp.sum(1) / r[:, 5], -(dp * dx * dx).sum(1) / 2, -(dp * dx * dy).sum(1), -(dp * dy * dy).sum(1) / 2,
                  (dp * (r[:, 2:3] * dx + r[:, 3:4] * dy)).sum(1), (dp * (r[:, 3:4] * dx + r[:, 4:5] * dy)).sum(1)]
        grad.index_add_(0, row, torch.stack(terms, 1))

    _walk(rec, lists, cam, TX, TY, gradients)
    full = torch.zeros((case["n"], 9), dtype=torch.float64, device="cuda")
    full[ids] = grad
    out = {"image": images[0], "rgb": full[:, :3], "opacity": full[:, 3], "conic": full[:, 4:7], "xy": full[:, 7:]}
    if case["precision"] != "fp32":
        out["t_final"] = _plane(T, cam, TX, TY)
    return out
