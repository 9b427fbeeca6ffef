"""What the compiler reports about the kernels of the built library: the metadata of every code object in liboctopus.so
(registers, scratch, LDS), by kernel.  Read on the CPU; nothing is run."""
import struct

import msgpack

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of the offload bundles in a shared library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + id_len]
            pos += 24 + id_len
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


def _metadata(elf):
    """The AMDGPU metadata notes (type 32) of a 64-bit little-endian ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entsize)
        if kind != 7:       # SHT_NOTE
            continue
        pos = offset
        while pos < offset + size:
            n_name, n_desc, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (n_name + 3) // 4 * 4
            if note == 32:
                yield msgpack.unpackb(elf[desc:desc + n_desc], raw=False, strict_map_key=False)
            pos = desc + (n_desc + 3) // 4 * 4


def kernels(path):
    """{mangled name: metadata} of every kernel in the library."""
    with open(path, "rb") as f:
        blob = f.read()
    return {k[".name"]: k for elf in _code_objects(blob) for m in _metadata(elf) for k in m["amdhsa.kernels"]}
