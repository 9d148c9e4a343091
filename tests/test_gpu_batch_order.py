"""Batches of more work items than the persistent launch has workgroups, whose jobs the launch takes in the
order of their items: every job's image equal to its own single launch, whatever the caller's order, for
the FP32 and tensorized rasterizers, tiles and groups."""
import numpy as np
import pytest

from paper_2605_17855_amd import gs, scenes
from gpu_helpers import note

pytestmark = pytest.mark.gpu

SIZES = [(1920, 1080), (16, 16), (1000, 700), (640, 360), (1000, 700)]
CASES = [("fp32", 1, 2), ("fp32", 2, 2), ("fp32", 4, 2), ("fp16", 1, 2), ("fp16", 2, 2), ("fp16", 4, 2), ("bf16", 1, 3),
         ("bf16", 8, 3)]


@pytest.mark.parametrize("tight", [False, True])
@pytest.mark.parametrize("prec,group,splits", CASES)
def test_large_batch_matches_single_images(prec, group, splits, tight):
    import torch
    note(f"batch order: {prec}, group {group}, culled {tight}")
    opt = gs.options(group=group, precision=prec, splits=splits, bg=(0.1, 0.2, 0.3), tight=tight,
                     aux_flags=gs.GS_AUX_NEVAL)
    frames = []
    for i, (w, h) in enumerate(SIZES):
        sc, cam = scenes.camera_box_scene(4000, seed=20 + i), scenes.pinhole(w, h, 60.0)
        r = gs.Renderer(sc.n, w, h, group=group)
        r.render(gs.DeviceScene(sc), cam, opt)
        torch.cuda.synchronize()
        frames.append((r, cam, r.image.clone(), r.aux.clone()))
    parts = 1 if group == 1 else 2 if group == 2 and prec != "fp32" else group * group
    items = sum(((w + 16 * group - 1) // (16 * group)) * ((h + 16 * group - 1) // (16 * group)) * parts for w, h in SIZES)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert items > 8 * cus
    counter = torch.zeros(gs.BATCH_COUNTER_WORDS, dtype=torch.int32, device="cuda")
    for order in (range(5), [4, 2, 0, 3, 1]):
        for noalloc in (False, True):
            jobs = [(frames[i][0].proj, frames[i][0].bins, frames[i][1], torch.full_like(frames[i][2], -1.0),
                     torch.full_like(frames[i][3], -1.0)) for i in order]
            if noalloc:
                gs.gs_rasterize_batch_noalloc(jobs, opt)
            else:
                gs.gs_rasterize_batch(jobs, opt, counter)
            torch.cuda.synchronize()
            for i, job in zip(order, jobs):
                assert torch.equal(job[3], frames[i][2]) and torch.equal(job[4], frames[i][3]), (i, list(order))
