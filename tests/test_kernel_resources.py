"""What the compiler made of the kernels with several lanes per region, read from
the kernel descriptors' notes in libgm.so: no per-lane array in scratch memory
(which an array indexed by the lane number becomes).  Scratch that holds nothing
but spilled registers, four bytes each, is a matter of tuning and not looked at
here."""
from __future__ import annotations

import os
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_01573_amd", "libgm.so")

NT_AMDGPU_METADATA, SHT_NOTE = 32, 7


def _code_objects(lib: bytes):
    at = lib.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (count,) = struct.unpack_from("<Q", lib, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", lib, entry)
            if b"gfx950" in lib[entry + 24:entry + 24 + length] and size:
                yield lib[at + offset:at + offset + size]
            entry += 24 + length
        at = lib.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf: bytes):
    (sections,) = struct.unpack_from("<Q", elf, 40)
    entsize, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        if struct.unpack_from("<I", elf, sections + k * entsize + 4)[0] != SHT_NOTE:
            continue
        at, size = struct.unpack_from("<QQ", elf, sections + k * entsize + 24)
        end = at + size
        while at < end:
            name, desc, kind = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if kind == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            at = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(LIB, "rb") as fh:
        lib = fh.read()
    return [k for elf in _code_objects(lib) for k in _kernels(elf)]


@pytest.mark.parametrize("name,least", [("rule_wpr_kernel", 270), ("factor_wpr_kernel", 90),
                                        ("rule9_kernel", 220), ("factor9_kernel", 35),
                                        ("rule_gk_kernel", 70)])
def test_no_scratch_array(kernels, name, least):
    found = [k for k in kernels if name in k[".name"]]
    assert len(found) >= least, (name, len(found), len(kernels))
    bad = [(k[".name"], k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in found
           if k[".private_segment_fixed_size"] > 4 * k[".vgpr_spill_count"] + 8]
    assert not bad, bad[:8]
