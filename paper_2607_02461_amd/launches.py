"""The kernels a library call launches, read off the call itself.

Which kernel serves a layer is the library's choice by sizes and bit widths, so a test of one kernel, and a
report that names kernels, ask for what ran instead of repeating the rule: the call is recorded into a HIP
graph (nothing executes) and the graph's kernel nodes are listed in the order of their launches.
"""

import ctypes
import re
from typing import NamedTuple, Tuple

import torch


class Launch(NamedTuple):
    kernel: str                    # as lut_gemm_kernel<4,3,true>
    grid: Tuple[int, int, int]     # workgroups
    block: Tuple[int, int, int]    # threads


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("blockDim", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("gridDim", _Dim3),
                ("kernelParams", ctypes.c_void_p), ("sharedMemBytes", ctypes.c_uint)]


_CAPTURE_RELAXED = 2
_NODE_KERNEL = 0


def _runtime() -> ctypes.CDLL:
    """The HIP runtime this process already uses."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "/libamdhip64.so" in line}
    if not paths:
        raise RuntimeError("the HIP runtime is not loaded")
    hip = ctypes.CDLL(sorted(paths)[0])
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    return hip


def short_name(mangled: str) -> str:
    """The kernel's own name and its integer and boolean template arguments, of an Itanium-mangled name
    (_ZN <length><identifier> ... I <arguments> E ...)."""
    word, at = mangled, 3 if mangled.startswith("_ZN") else 2
    while (m := re.compile(r"\d+").match(mangled, at)):
        at = m.end() + int(m.group())
        word = mangled[m.end():at]
    args = re.compile(r"I((?:L[bij]n?\d+E)+)E").match(mangled, at)
    if not args:
        return word
    vals = re.findall(r"L([bij])(n?\d+)E", args.group(1))
    return f"{word}<{','.join(('false', 'true')[int(v)] if t == 'b' else v.replace('n', '-') for t, v in vals)}>"


def launches(call) -> list:
    """The kernel launches that `call()` enqueues on torch's current stream.  The call is captured, not run: its
    outputs keep their contents, so it is given outputs that exist (a tensor it creates is never written)."""
    hip = _runtime()

    def ok(status, what):
        if status:
            raise RuntimeError(f"{what} failed with HIP error {status}")

    stream = torch.cuda.Stream()
    graph = ctypes.c_void_p()
    with torch.cuda.stream(stream):
        handle = ctypes.c_void_p(stream.cuda_stream)
        ok(hip.hipStreamBeginCapture(handle, _CAPTURE_RELAXED), "hipStreamBeginCapture")
        try:
            call()
        finally:
            ended = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
        ok(ended, "hipStreamEndCapture")
    try:
        n = ctypes.c_size_t(0)
        ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)), "hipGraphGetNodes")
        nodes = (ctypes.c_void_p * max(1, n.value))()
        ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)), "hipGraphGetNodes")
        out = []
        for node in list(nodes)[:n.value]:
            kind = ctypes.c_int(-1)
            ok(hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)), "hipGraphNodeGetType")
            if kind.value != _NODE_KERNEL:
                raise RuntimeError(f"the call records a graph node of type {kind.value}, not a kernel")
            p = _KernelNodeParams()
            ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)), "hipGraphKernelNodeGetParams")
            name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), handle)
            if not name:
                raise RuntimeError("a captured kernel has no name")
            out.append(Launch(short_name(name.decode()), (p.gridDim.x, p.gridDim.y, p.gridDim.z),
                              (p.blockDim.x, p.blockDim.y, p.blockDim.z)))
        return out
    finally:
        hip.hipGraphDestroy(graph)
