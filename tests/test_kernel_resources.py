"""Every kernel keeps its values in registers: the code objects in the built library ask for no scratch memory (a reload from it
waits for all loads that are in flight, rows fetched ahead among them).  Reads the metadata notes, needs no GPU."""
import os
import struct

import pytest

from paper_2503_10325_amd import binding as sv

msgpack = pytest.importorskip("msgpack")
pytestmark = pytest.mark.skipif(not os.path.exists(sv.LIB_PATH), reason="libspecverify.so not built")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The device ELF images of all bundles: (count, then offset, size and name of each entry) behind the magic."""
    at = data.find(MAGIC)
    while at >= 0:
        count, pos = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, pos)
            if b"amdgcn" in data[pos + 24:pos + 24 + name] and size:
                yield data[at + offset:at + offset + size]
            pos += 24 + name
        at = data.find(MAGIC, at + 1)


def kernels(elf):
    """amdhsa.kernels of the AMDGPU metadata note (type 32)."""
    sections, entry, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, offset, size = struct.unpack_from("<I16xQQ", elf, sections + i * entry + 4)
        end = offset + size
        while kind == 7 and offset < end:
            name, desc, note = struct.unpack_from("<III", elf, offset)
            body = offset + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            offset = body + (desc + 3) // 4 * 4


def test_no_kernel_uses_scratch_memory():
    with open(sv.LIB_PATH, "rb") as f:
        found = [k for elf in code_objects(f.read()) for k in kernels(elf)]
    assert len(found) > 50
    bad = [(k[".name"], k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in found
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]
    assert not bad
