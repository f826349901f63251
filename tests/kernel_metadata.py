"""Metadata of the kernels built into libtpo.so (registers, wavefront size), read from the code objects'
AMDGPU notes; no GPU needed."""
import struct

import msgpack

from paper_2604_19906_amd import tpo

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + idlen]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + idlen
        at = blob.find(MAGIC, pos)


def _notes(elf):
    """Descriptors of the ELF64 file's notes (NT_AMDGPU_METADATA = 32)."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phentsize)
        if kind != 4:                                   # PT_NOTE
            continue
        pos = offset
        while pos < offset + size:
            namesz, descsz, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (namesz + 3) // 4 * 4
            if note == 32:
                yield elf[desc:desc + descsz]
            pos = desc + (descsz + 3) // 4 * 4


def kernels():
    """Mangled kernel name -> its metadata (``.vgpr_count``, ``.agpr_count``, ...)."""
    with open(tpo.LIB_PATH, "rb") as f:
        blob = f.read()
    return {k[".name"]: k for elf in _code_objects(blob) for desc in _notes(elf)
            for k in msgpack.unpackb(desc)["amdhsa.kernels"]}
