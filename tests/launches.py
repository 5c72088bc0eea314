"""The kernels that calls on a stream launch, by name: recorded in a graph
capture (nothing runs) and read from its nodes."""
import ctypes


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("blockDim", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("gridDim", _Dim3), ("kernelParams", ctypes.c_void_p), ("sharedMemBytes", ctypes.c_uint32)]


def recorded(stream, f):
    """mangled names of the kernels that f launches on the torch stream, in
    the order they were recorded"""
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    s, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)

    def ok(r):
        assert r == 0, r
    ok(hip.hipStreamBeginCapture(s, 1))                 # thread-local mode
    f()
    ok(hip.hipStreamEndCapture(s, ctypes.byref(graph)))
    ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
    nodes = (ctypes.c_void_p * n.value)()
    ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
    names = []
    for node in nodes:
        kind, p = ctypes.c_int(-1), _KernelNodeParams()
        ok(hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)))
        assert kind.value == 0                          # a kernel
        ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)))
        names.append(hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), s).decode())
    ok(hip.hipGraphDestroy(graph))
    return names
