"""Registers of the built kernels, from the metadata of the library's own code
objects: what a kernel cannot hold in registers it keeps in memory, on every
use. Queries and forward passes of the default shapes have no such spills, but
for FP32 queries with four features, whose gathers alone take 64 registers, and
four registers of a grouped query."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_16237_amd", "libnbvh.so")


def _code_objects(data):
    """The gfx950 code objects of the offload bundles in a host library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24: p + 24 + name]:
                yield data[at + off: at + off + size]
            p += 24 + name
        at += 24


def _kernels(obj):
    """amdhsa.kernels of a code object (the ELF note of type 32)."""
    sections, = struct.unpack_from("<Q", obj, 40)
    entry, count = struct.unpack_from("<HH", obj, 58)
    for i in range(count):
        if struct.unpack_from("<I", obj, sections + i * entry + 4)[0] != 7:
            continue
        p, size = struct.unpack_from("<QQ", obj, sections + i * entry + 24)
        end = p + size
        while p < end:
            name, desc, kind = struct.unpack_from("<III", obj, p)
            p += 12 + (name + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(obj[p: p + desc], strict_map_key=False)["amdhsa.kernels"]
            p += (desc + 3) // 4 * 4


def _spills():
    with open(LIB, "rb") as f:
        data = f.read()
    return {k[".name"]: k[".vgpr_spill_count"] for obj in _code_objects(data) for k in _kernels(obj)}


def test_default_queries_and_forward_passes_do_not_spill():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    spills = _spills()
    # default shape: eight waves, two levels at a time, no pair or LDS gathers
    default = re.compile(r"k_query_eval(_batch)?I.*ELi8ELi2ELi0E|k_query_smallI|k_forwardI")
    seen = {n: s for n, s in spills.items() if default.search(n)}
    assert len(seen) == 24  # four kernels, three precisions, two feature counts
    wide = re.compile(r"IfLi4E")  # FP32, four features
    assert max(s for n, s in seen.items() if wide.search(n)) <= 24
    rest = {n: s for n, s in seen.items() if s and not wide.search(n)}
    assert {n: s for n, s in rest.items() if "_batch" not in n} == {}
    assert all(s <= 4 for s in rest.values())  # grouped queries
    assert all(s == 0 for n, s in seen.items() if "k_forward" in n)
