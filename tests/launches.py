"""Which kernels a call launches, and with what grid: the call is recorded into a
graph, whose kernel nodes are read back."""

import ctypes

import torch


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class _KernelParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _hip():
    with open("/proc/self/maps") as f:  # the runtime this process already uses
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    hip = ctypes.CDLL(sorted(paths)[0])
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    return hip


def captured(call):
    """[(kernel name, workgroups, threads)] of the kernels `call` enqueues on the current stream, in order."""
    call()  # device properties are asked for once per process, before the recording
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip = _hip()
    raw = ctypes.c_void_p(graph.raw_cuda_graph())
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    out = []
    for node in nodes:
        p = _KernelParams()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        name = hip.hipKernelNameRefByPtr(p.func, None).decode()
        out.append((name, p.grid.x, p.block.x))
    return out
