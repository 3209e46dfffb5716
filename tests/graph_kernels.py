"""The kernels that a call enqueues, as (name, blocks): the call is captured
into a HIP graph (nothing runs) and the graph's kernel nodes are read.  Tests
use it to assert which kernel the dispatch took, where results alone cannot
tell."""

import ctypes
import re

import torch


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):          # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


_hip = None


def _runtime():
    """The HIP runtime that this process has loaded."""
    global _hip
    if _hip is None:
        with open("/proc/self/maps") as f:
            path = next(line.split()[-1] for line in f if re.search(r"/libamdhip64\.so[.\d]*$", line.rstrip()))
        _hip = ctypes.CDLL(path)
        _hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
        _hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        _hip.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
        _hip.hipGraphNodeGetType.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_int)]
        _hip.hipGraphKernelNodeGetParams.argtypes = [ctypes.c_void_p, ctypes.POINTER(_KernelNodeParams)]
    return _hip


def kernels(fn):
    """[(mangled kernel name, blocks)] of the kernels fn() enqueues on the current stream."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        fn()
    hip, raw = _runtime(), ctypes.c_void_p(g.raw_cuda_graph())
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    out = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(node, ctypes.byref(kind)) == 0
        if kind.value != 0:                         # hipGraphNodeTypeKernel
            continue
        p = _KernelNodeParams()
        assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(p)) == 0
        out.append((hip.hipKernelNameRefByPtr(p.func, None).decode(), p.grid.x))
    return out


def lanes(name):
    """Lanes per element of a drelu / relu / replicated-sharing kernel, by its (mangled) name."""
    m = re.search(r"k_drelu_wavesI.*?Lb[01]ELi([24])EE", name)
    if m:
        return int(m.group(1))
    if "k_rss_wavesI" in name:
        return 4
    assert re.search(r"\dk_(drelu|rss)I", name), name
    return 1
