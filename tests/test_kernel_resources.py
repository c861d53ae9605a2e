"""Registers of the built kernels, from the metadata that the compiler wrote into
libedm.so: none spills (a spill in a scan or a walk is memory traffic on its
inner path, and scratch for a kernel is allocated at its first launch), and the
exact scans hold the waves that the choice of their workgroups counts with."""
from __future__ import annotations

import re
import struct

import msgpack
import pytest

from paper_2105_12301_amd import edm

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length]:
                yield blob[at + off:at + off + size]
            p += 24 + length
        at = blob.find(MAGIC, at + 1)


def _notes(elf):
    (sections,) = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        (kind,) = struct.unpack_from("<I", elf, sections + i * size + 4)
        at, length = struct.unpack_from("<QQ", elf, sections + i * size + 0x18)
        end = at + length
        while kind == 7 and at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            data = at + 12 + (name + 3) // 4 * 4
            if note == 32:  # AMDGPU metadata
                yield msgpack.unpackb(elf[data:data + desc], raw=False, strict_map_key=False)
            at = data + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(edm.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for e in _code_objects(blob) for m in _notes(e) for k in m["amdhsa.kernels"]}
    assert len(found) > 300
    return found


def test_no_kernel_uses_scratch(kernels):
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in kernels.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad


def test_exact_scans_hold_the_waves_they_are_launched_for(kernels):
    seen = 0
    for name, k in kernels.items():
        # k_knn<E, k, lag 1, waves, 1 (no split), queued>
        m = re.search(r"k_knnILi(\d+)ELi\d+ELb[01]ELi(?:4|8|16)ELi1E", name)
        if not m or m.group(1) == "0":
            continue
        E = int(m.group(1))
        most = 64 if E <= 6 else 80 if E <= 9 else 96 if E <= 11 else 128 if E <= 16 else 168
        assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= most, (name, k[".vgpr_count"])
        seen += 1
    assert seen >= 80
