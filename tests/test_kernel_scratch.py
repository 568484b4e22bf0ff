"""A kernel that needs scratch memory has the runtime set it aside on a queue's
first launch of it.  The allocation-free tick's kernels need none: read from
the resource metadata of the code objects in the built library."""
from __future__ import annotations

import os
import struct

import pytest

from paper_1906_02318_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(blob):
    """The GPU code objects of the library's offload bundles (64-bit ELF images)."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", blob, p)
            target = blob[p + 24:p + 24 + name]
            p += 24 + name
            if b"amdgcn" in target:
                yield blob[at + offset:at + offset + size]
        at += len(magic)


def _kernels(elf):
    """The kernels of a code object's metadata note (type 32), each a dict."""
    (sections,) = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        at = sections + k * entry
        if struct.unpack_from("<I", elf, at + 4)[0] != 7:  # SHT_NOTE
            continue
        p, size = struct.unpack_from("<QQ", elf, at + 24)
        end = p + size
        while p < end:
            name, desc, kind = struct.unpack_from("<III", elf, p)
            p += 12 + (name + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(elf[p:p + desc])["amdhsa.kernels"]
            p += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    return [k for elf in _code_objects(blob) for k in _kernels(elf)]


@pytest.mark.parametrize("name", ["tick_fp32_kernel", "tick_split_kernel", "tick_custom_split_kernel",
                                  "recheck64_filter_kernel", "recheck64_kernel", "recheck64_rc_kernel"])
def test_the_allocation_free_ticks_kernels_need_no_scratch(kernels, name):
    mine = [k for k in kernels if f"mpmi{len(name)}{name}" in k[".name"]]
    assert mine
    assert {k[".name"]: k[".private_segment_fixed_size"] for k in mine if k[".private_segment_fixed_size"]} == {}
