"""What the compiler says about the kernels of the built library: the metadata of its gfx950 code objects, read from the file."""
import os
import struct

import msgpack

from paper_2111_14255_amd import build


def objects():
    """The gfx950 code objects (ELF images) of the library's offload bundles."""
    data = open(os.environ.get("MTSCHED_LIB") or build.lib_path(), "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<3Q", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if size and b"gfx950" in target:
                yield data[at + offset:at + offset + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)


def kernels():
    """Metadata of every kernel, by mangled name."""
    out = {}
    for elf in objects():
        headers, = struct.unpack_from("<Q", elf, 32)
        n, = struct.unpack_from("<H", elf, 56)
        for i in range(n):
            kind, _, offset = struct.unpack_from("<IIQ", elf, headers + 56 * i)
            if kind != 4:                                    # PT_NOTE
                continue
            name, size, note = struct.unpack_from("<III", elf, offset)
            if note == 32:                                   # NT_AMDGPU_METADATA
                at = offset + 12 + (name + 3) // 4 * 4
                out.update({k[".name"]: k for k in msgpack.unpackb(elf[at:at + size], strict_map_key=False)["amdhsa.kernels"]})
    return out


def held_by_registers(kernel):
    """Workgroups of a kernel whose registers a compute unit holds: 512 per lane of each of four SIMDs, given out in eights."""
    waves = kernel[".max_flat_workgroup_size"] // 64
    return 512 // ((kernel[".vgpr_count"] + 7) // 8 * 8) * 4 // waves
