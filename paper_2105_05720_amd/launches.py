"""Which kernels a call launches, read from a HIP graph that captures it: nothing is executed, and nothing is derived from the
library's rules a second time.  A measurement and test aid."""
from __future__ import annotations

import ctypes as C
import re
from typing import Callable, List, NamedTuple

import torch


class Launch(NamedTuple):
    kernel: str          # name without namespace and arguments
    symbol: str          # the mangled name, template arguments included
    grid: int            # workgroups
    block: int           # threads of each


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNodeParams(C.Structure):       # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p), ("shared", C.c_uint32)]


def _runtime() -> C.CDLL:
    """The HIP runtime that torch has loaded."""
    with open("/proc/self/maps") as maps:
        for line in maps:
            if "libamdhip64" in line:
                return C.CDLL(line.split()[-1])
    raise RuntimeError("the HIP runtime is not loaded")


def launches(call: Callable[[], None]) -> List[Launch]:
    """The kernels that `call` enqueues on the current stream, in order."""
    hip = _runtime()
    hip.hipKernelNameRefByPtr.restype = C.c_char_p

    def check(rc):
        if rc != 0:
            raise RuntimeError("HIP error %d while reading a captured graph" % rc)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call()
    raw, n = C.c_void_p(graph.raw_cuda_graph()), C.c_size_t()
    check(hip.hipGraphGetNodes(raw, None, C.byref(n)))
    nodes = (C.c_void_p * n.value)()
    check(hip.hipGraphGetNodes(raw, nodes, C.byref(n)))
    out = []
    for node in nodes:
        kind, p = C.c_int(), _KernelNodeParams()
        check(hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)))
        if kind.value != 0:                 # hipGraphNodeTypeKernel
            out.append(Launch("node of type %d" % kind.value, "", 0, 0))
            continue
        check(hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)))
        symbol = (hip.hipKernelNameRefByPtr(C.c_void_p(p.func), None) or b"?").decode()
        named = re.match(r"_ZN3ccfL?(\d+)(\w+)", symbol)
        out.append(Launch(named.group(2)[:int(named.group(1))] if named else symbol, symbol, p.grid.x, p.block.x))
    return out
