"""Register use of the built kernels, from the metadata of the code objects in
the shared library: a kernel that holds its matrix in registers and spills it
is many times slower, with the same results."""

import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1612_07875_amd", "libdmdstream.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """AMDGPU metadata maps of one code object (the ELF64 note sections)."""
    shoff = struct.unpack_from("<Q", elf, 0x28)[0]
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        typ, off, size = struct.unpack_from("<4xI16xQQ", elf, shoff + i * shentsize)
        at, end = off, off + size
        while typ == 7 and at + 12 <= end:
            nlen, dlen, kind = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (nlen + 3) // 4 * 4
            if elf[at + 12:at + 12 + nlen].rstrip(b"\0") == b"AMDGPU" and kind == 32:
                yield msgpack.unpackb(elf[desc:desc + dlen], strict_map_key=False)
            at = desc + (dlen + 3) // 4 * 4


def _kernels():
    with open(LIB, "rb") as f:
        data = f.read()
    out, at = {}, data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        count = struct.unpack_from("<Q", data, pos)[0]
        pos += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            ident = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"amdgcn" in ident and size:
                for note in _notes(data[at + off:at + off + size]):
                    for k in note["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at = data.find(MAGIC, at + len(MAGIC))
    return out


def test_registers_are_not_spilled():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    kernels = _kernels()
    assert len(kernels) > 50, "no kernel metadata found"
    # the largest reduction holds 192 registers of matrix per lane and spills
    # 11 others; a matrix that is spilled costs a hundred and more
    spills = {n: k[".vgpr_spill_count"] for n, k in kernels.items() if k.get(".vgpr_spill_count", 0) > 32}
    assert not spills, spills
