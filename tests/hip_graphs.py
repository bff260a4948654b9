"""Graph capture through the HIP runtime itself: what a capture recorded, and replays of it."""
import ctypes as C
import re

import torch


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNodeParams(C.Structure):
    _fields_ = [("blockDim", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("gridDim", _Dim3),
                ("kernelParams", C.c_void_p), ("sharedMemBytes", C.c_uint32)]


_hip = None


def hip():
    """The runtime library that torch (and libsp.so) have loaded."""
    global _hip
    if _hip is None:
        torch.cuda.init()
        path = re.search(r"\S*libamdhip64\S*", open("/proc/self/maps").read()).group(0)
        _hip = C.CDLL(path)
    return _hip


def _ok(err):
    assert err == 0, "HIP error %d" % err


class Graph:
    """What `work` enqueues on `stream` (a torch stream), captured."""

    def __init__(self, stream, work):
        self.stream, self.graph, self.exec_ = stream, C.c_void_p(), C.c_void_p()
        s = C.c_void_p(stream.cuda_stream)
        _ok(hip().hipStreamBeginCapture(s, 0))           # global mode, the strictest
        try:
            work()
        finally:
            err = hip().hipStreamEndCapture(s, C.byref(self.graph))
        _ok(err)

    def grids(self):
        """(x, y, z) of every kernel launch"""
        n = C.c_size_t(0)
        _ok(hip().hipGraphGetNodes(self.graph, None, C.byref(n)))
        nodes = (C.c_void_p * n.value)()
        _ok(hip().hipGraphGetNodes(self.graph, nodes, C.byref(n)))
        out = []
        for node in nodes:
            kind, p = C.c_int(-1), _KernelNodeParams()
            _ok(hip().hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)))
            assert kind.value == 0, "a node that is no kernel: type %d" % kind.value
            _ok(hip().hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)))
            out.append((p.gridDim.x, p.gridDim.y, p.gridDim.z))
        return out

    def replay(self, stream=None):
        if not self.exec_:
            _ok(hip().hipGraphInstantiate(C.byref(self.exec_), self.graph, None, None, C.c_size_t(0)))
        _ok(hip().hipGraphLaunch(self.exec_, C.c_void_p((stream or self.stream).cuda_stream)))

    def destroy(self):
        if self.exec_:
            _ok(hip().hipGraphExecDestroy(self.exec_))
        _ok(hip().hipGraphDestroy(self.graph))
