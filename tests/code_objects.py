"""The gfx950 code objects inside the built library, and what their metadata says of each kernel."""

import os
import struct

import msgpack

import paper_2607_02461_amd as oq
from paper_2607_02461_amd.launches import short_name

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_NT_AMDGPU_METADATA = 32


def code_objects():
    """The device ELF images, one per source file with kernels."""
    with open(oq.LIB_PATH, "rb") as f:
        data = f.read()
    out, at = [], data.find(_MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(entries):
            offset, size, name_len = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + name_len]
            p += 24 + name_len
            if size and name.endswith(b"gfx950"):
                out.append(data[at + offset:at + offset + size])
        at = data.find(_MAGIC, at + len(_MAGIC))
    assert out, f"{os.path.basename(oq.LIB_PATH)} holds no gfx950 code objects"
    return out


def kernel_metadata():
    """{kernel as lut_gemm_wave<4,4,2,4,2>: its metadata map}."""
    kernels = {}
    for elf in code_objects():
        shoff, = struct.unpack_from("<Q", elf, 40)
        shentsize, shnum = struct.unpack_from("<HH", elf, 58)
        for i in range(shnum):
            kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
            offset, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
            if kind != 7:   # SHT_NOTE
                continue
            p = offset
            while p < offset + size:
                name_size, desc_size, note = struct.unpack_from("<III", elf, p)
                desc = p + 12 + (name_size + 3) // 4 * 4
                if note == _NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(elf[desc:desc + desc_size])["amdhsa.kernels"]:
                        kernels[short_name(k[".name"])] = k
                p = desc + (desc_size + 3) // 4 * 4
    return kernels
