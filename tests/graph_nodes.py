"""The kernels a call launches, read from a HIP graph captured from it (nothing
is run): which route a dispatch takes, and the device memory it hands its
kernels."""

import ctypes

import torch


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class _KernelNodeParams(ctypes.Structure):   # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.POINTER(ctypes.c_void_p)), ("lds", ctypes.c_uint)]


def _hip():
    """The HIP runtime this process already uses."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64.so" in line}
    assert len(paths) == 1, paths
    hip = ctypes.CDLL(paths.pop())
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    return hip


class Kernel:
    def __init__(self, name, params, graph):
        self.name, self._params, self._graph = name, params, graph

    def pointer(self, i):
        """Argument i as an address."""
        return ctypes.c_uint64.from_address(self._params[i]).value


def capture(call):
    """A torch graph captured from call(), kept so that it can be replayed too."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    return g


def kernels(graph):
    """The kernel nodes of a captured graph."""
    hip, handle, n = _hip(), ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        kind, p = ctypes.c_int(), _KernelNodeParams()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value != 0:   # hipGraphNodeTypeKernel
            continue
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        name = hip.hipKernelNameRefByPtr(p.func, None)
        out.append(Kernel(name.decode(), p.params, graph))
    return out


def kernel_names(call):
    return [k.name for k in kernels(capture(call))]
