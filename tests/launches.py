"""Which kernels a call launches: the call is captured into a graph, which is never run, and the graph's kernel nodes are read."""
import ctypes
import re
import subprocess

import torch


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class _KernelNodeParams(ctypes.Structure):           # hipKernelNodeParams
    _fields_ = [("blockDim", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("gridDim", _Dim3),
                ("kernelParams", ctypes.c_void_p), ("sharedMemBytes", ctypes.c_uint)]


_KERNEL_NODE = 0                                     # hipGraphNodeTypeKernel


def _runtime():
    """The HIP runtime that torch and libnova.so share, already loaded."""
    with open("/proc/self/maps") as maps:
        paths = {ln.split()[-1] for ln in maps if "libamdhip64" in ln}
    assert len(paths) == 1, paths
    hip = ctypes.CDLL(paths.pop())
    vp = ctypes.c_void_p
    hip.hipGraphGetNodes.argtypes = [vp, ctypes.POINTER(vp), ctypes.POINTER(ctypes.c_size_t)]
    hip.hipGraphNodeGetType.argtypes = [vp, ctypes.POINTER(ctypes.c_int)]
    hip.hipGraphKernelNodeGetParams.argtypes = [vp, ctypes.POINTER(_KernelNodeParams)]
    hip.hipKernelNameRefByPtr.argtypes = [vp, vp]
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    return hip


def launches(call):
    """[(kernel with its template arguments, workgroups, threads of one)] in the order of the launches.  The call must allocate nothing
    (workspace and y are passed in)."""
    hip, graph = _runtime(), torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    handle, count = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(count)) == 0
    found = []
    for node in nodes:
        kind, params = ctypes.c_int(), _KernelNodeParams()
        assert hip.hipGraphNodeGetType(node, ctypes.byref(kind)) == 0
        assert kind.value == _KERNEL_NODE, kind.value
        assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(params)) == 0
        found.append((hip.hipKernelNameRefByPtr(params.func, None).decode(), params.gridDim.x, params.blockDim.x))
    names = "\n".join(name.replace("DF16_", "Dh") for name, _, _ in found)
    plain = subprocess.run(["c++filt"], input=names, capture_output=True, text=True, check=True).stdout.splitlines()
    plain = [re.search(r"(\w+<.*?>)\(", p)[1].replace("false", "0").replace("true", "1") for p in plain]
    return [(name, blocks, threads) for name, (_, blocks, threads) in zip(plain, found, strict=True)]
