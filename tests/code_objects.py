"""The gfx950 code objects inside the built library: what their metadata says of each kernel, and their code."""

import os
import re
import struct
import subprocess
import tempfile

import msgpack

import paper_2607_02461_amd as oq
from paper_2607_02461_amd.launches import short_name

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_NT_AMDGPU_METADATA = 32
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


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


def disassembly():
    """{kernel: its instructions as (mnemonic, operands) pairs in the order of the code}."""
    out = {}
    for elf in code_objects():
        with tempfile.NamedTemporaryFile(suffix=".elf") as f:
            f.write(elf)
            f.flush()
            text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", f.name], check=True,
                                  capture_output=True, text=True).stdout
        for line in text.splitlines():
            label = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if label:
                body = out.setdefault(short_name(label.group(1)), [])
            elif line.startswith("\t"):
                name, _, operands = line.split("//")[0].strip().partition(" ")
                body.append((name, [o.strip() for o in operands.split(", ")]))
    return out


def registers(operand):
    """The vector registers of an operand: v3, v[4:7], a[0:3] (accumulation registers from 1000 on)."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    base = 1000 if m[1] == "a" else 0
    return set(range(base + lo, base + hi + 1))


def mfma_hazards(code, before=2, after=11):
    """The places of `code` (as disassembly() gives it) where an MFMA reads registers that a VALU instruction wrote
    fewer than `before` wait states earlier, or another vector instruction touches registers that an MFMA
    writes fewer than `after` wait states earlier.  Along the code as it stands, branches not followed."""
    found, valu, mfma, now = [], {}, {}, 0   # register -> first wait state after the instruction that wrote it
    for at, (name, operands) in enumerate(code):
        regs = [registers(o) for o in operands]
        if name.startswith("v_mfma"):
            late = [r for o in regs[1:] for r in o if now - valu.get(r, -before) < before]
            mfma.update((r, now + 1) for r in regs[0])
        else:
            touched = set().union(*regs) if name.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")) else set()
            late = [r for r in touched if now - mfma.get(r, -after) < after]
            if name.startswith("v_"):
                swaps = "swap" in name
                valu.update((r, now + 1) for o in (regs if swaps else regs[:1]) for r in o)
        if late:
            found.append(f"{at}: {name} {', '.join(operands)}: registers {sorted(late)}")
        now += int(operands[0], 0) + 1 if name == "s_nop" else 1
    return found
