"""What the compiler made of the kernels, from the metadata of the built library's gfx950
code objects: no kernel keeps vector registers in scratch memory (each such access is a
wait for all loads in flight), and none asks for scratch memory at all (which the first
launch on a stream waits for, 240 us)."""
import struct

import pytest

import paper_0910_1517_amd as corr
from paper_0910_1517_amd import build

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels():
    corr.lib()
    data = open(build.LIB, "rb").read()
    pos = data.find(MAGIC)
    while pos >= 0:
        count, p = struct.unpack_from("<Q", data, pos + len(MAGIC))[0], pos + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + name_len]
            p += 24 + name_len
            if b"gfx950" in name:
                yield from metadata(data[pos + offset:pos + offset + size])
        pos = data.find(MAGIC, pos + 1)


def metadata(elf):
    """The kernels of the NT_AMDGPU_METADATA notes of a code object."""
    start = struct.unpack_from("<Q", elf, 40)[0]
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        header = start + i * size
        if struct.unpack_from("<I", elf, header + 4)[0] != 7:  # SHT_NOTE
            continue
        q, length = struct.unpack_from("<QQ", elf, header + 24)
        end = q + length
        while q < end:
            name_size, desc_size, kind = struct.unpack_from("<III", elf, q)
            q += 12 + (name_size + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(elf[q:q + desc_size])["amdhsa.kernels"]
            q += (desc_size + 3) // 4 * 4


def test_no_kernel_spills_vector_registers():
    found = list(kernels())
    assert any("xengine_kernel" in k[".name"] for k in found) and len(found) > 100
    assert [k[".name"] for k in found if k[".vgpr_spill_count"]] == []
    assert [k[".name"] for k in found if k[".private_segment_fixed_size"]] == []
