"""Every workgroup barrier of the raster, backward and block expansion kernels waits for the wave's own LDS
writes first: in the gfx950 code, no path of straight-line instructions leads from an LDS write
to a barrier, and no barrier heads a block, without `lgkmcnt(0)` between (the compiler was
seen to leave the wait out at barriers in loop headers, for writes pending over the back edge)."""
import os
import re
import subprocess

import pytest

from paper_2605_17855_amd import build


def _unwaited(asm: str):
    bad, fn = [], ""
    lines = [x.strip() for x in asm.split("\n")]
    for i, ln in enumerate(lines):
        if re.match(r"^_Z\w+:", ln):
            fn = ln.split(":")[0]
        if not ln.startswith("s_barrier"):
            continue
        for prev in reversed(lines[:i]):
            if not prev or prev.startswith(";"):
                continue
            if "lgkmcnt(0)" in prev:
                break
            if re.match(r"^ds_(write|add|max|min|or|and)", prev) or prev.split(";")[0].strip().endswith(":"):
                bad.append((fn, i + 1))
                break
    return bad


def test_scan_finds_a_missing_wait():
    """The scan itself: a write before a barrier, a barrier at a block's head, a waited one."""
    assert _unwaited("_Zf:\n s_waitcnt lgkmcnt(0)\n ds_write_b32 v0, v1\n s_barrier") == [("_Zf", 4)]
    assert _unwaited("_Zf:\n v_nop\n.LBB0_1:\n v_nop\n s_barrier") == [("_Zf", 5)]
    assert _unwaited("_Zf:\n ds_write_b32 v0, v1\n s_waitcnt vmcnt(0) lgkmcnt(0)\n s_barrier") == []


@pytest.mark.parametrize("source", ["gs_raster_fp32.hip", "gs_raster_mfma.hip", "gs_backward.hip", "gs_blocks.hip"])
def test_barriers_wait_for_lds_writes(source, tmp_path):
    out = tmp_path / "k.s"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-c",
                        os.path.join(build.CSRC, source), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    asm = out.read_text()
    assert "s_barrier" in asm
    assert _unwaited(asm) == []


@pytest.mark.parametrize("source", ["gs_sort.hip", "gs_preprocess.hip"])
def test_barriers_of_sorts_and_scans_wait_for_lds_writes(source, tmp_path):
    test_barriers_wait_for_lds_writes(source, tmp_path)


def test_every_source_with_barriers_is_scanned():
    scanned = {"gs_raster_fp32.hip", "gs_raster_mfma.hip", "gs_backward.hip", "gs_blocks.hip", "gs_sort.hip",
               "gs_preprocess.hip"}
    for source in build.SOURCES:
        with open(os.path.join(build.CSRC, source)) as f:
            assert source in scanned or not re.search(r"block_sync|__syncthreads", f.read()), source
