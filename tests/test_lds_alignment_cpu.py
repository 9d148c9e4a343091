"""LDS arrays that the kernels access in wider units than their elements are declared with that
alignment: left to the compiler's layout of LDS, a 32-bit store into an array of 16-bit counters may or
may not be aligned."""
import os
import re

import pytest

from paper_2605_17855_amd import build

SIZE = {"uint8_t": 1, "bool": 1, "uint16_t": 2, "short": 2, "ushort2": 4, "uint32_t": 4, "int": 4, "float": 4,
        "uint64_t": 8, "float2": 8, "uint2": 8, "short8": 16, "ushort4": 8, "double": 8, "double2": 16, "float4": 16,
        "float4v": 16, "uint4": 16}
ARRAY = re.compile(r"(__shared__\s+)?(?:__align__\((\d+)\)\s*)?\b(\w+)\s+(\w+)((?:\[[^\]]+\])+)\s*;")
CAST = re.compile(r"reinterpret_cast<(?:const\s+)?(?:\w+::)?(\w+)\s*\*>\(\s*&?((?:\w+\.)*)(\w+)\[")


def _bad(source: str):
    """(array, element, unit) of every wider access to a too weakly aligned LDS array: a __shared__ one, or a
    member reached through a struct."""
    local, member = {}, {}
    for m in ARRAY.finditer(source):
        shared, align, elem, name, _ = m.groups()
        if elem in SIZE:
            (local if shared else member).setdefault(name, []).append((m.start(), elem, max(int(align or 0), SIZE[elem])))
    bad = []
    for m in CAST.finditer(source):
        unit, owner, name = m.groups()
        # a kernel's own array: its last declaration before; a name of several structs: the strongest one
        decl = member.get(name, []) if owner else [d for d in local.get(name, []) if d[0] < m.start()][-1:]
        if decl:
            _, elem, align = max(decl, key=lambda d: d[2])
            if SIZE.get(unit, 1) > align:
                bad.append((name, elem, unit))
    return bad


def test_scan_finds_a_weak_array():
    text = "__shared__ %suint16_t n[4][256];\n reinterpret_cast<uint32_t *>(&n[0][0])[i] = 0;"
    assert _bad(text % "") == [("n", "uint16_t", "uint32_t")] and _bad(text % "__align__(16) ") == []
    text = "struct S { %suint32_t c[2][4]; };\n x = *reinterpret_cast<const uint4 *>(sm.c[i]);"
    assert _bad(text % "") == [("c", "uint32_t", "uint4")] and _bad(text % "__align__(16) ") == []


@pytest.mark.parametrize("source", build.SOURCES + build.HEADERS)
def test_wider_accesses_are_aligned(source):
    with open(os.path.join(build.CSRC, source)) as f:
        assert _bad(f.read()) == []
