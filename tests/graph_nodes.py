"""The kernel nodes that a call records into a HIP graph: their grids and
workgroups, read back without running them."""

import ctypes


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("blockDim", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("gridDim", _Dim3), ("kernelParams", ctypes.c_void_p),
                ("sharedMemBytes", ctypes.c_uint32)]


def _hip():
    maps = open("/proc/self/maps").read()
    return ctypes.CDLL(next(line.split()[-1] for line in maps.splitlines()
                            if "libamdhip64" in line))


def _ok(status):
    assert status == 0, f"HIP status {status}"


def kernel_nodes(call):
    """[(workgroups, threads per workgroup)] of the kernels that call(stream)
    records on a capturing stream, in no particular order; nothing is run."""
    import torch
    hip, graph, n = _hip(), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    stream = ctypes.c_void_p(side.cuda_stream)
    _ok(hip.hipStreamBeginCapture(stream, 1))        # thread-local mode
    try:
        call(side)
    finally:
        end = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
    _ok(end)
    try:
        _ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
        nodes = (ctypes.c_void_p * n.value)()
        _ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
        out = []
        for node in nodes:
            kind, p = ctypes.c_int(), _KernelNodeParams()
            node = ctypes.c_void_p(node)
            _ok(hip.hipGraphNodeGetType(node, ctypes.byref(kind)))
            assert kind.value == 0, "a kernel node"
            _ok(hip.hipGraphKernelNodeGetParams(node, ctypes.byref(p)))
            out.append((p.gridDim.x, p.blockDim.x))
        return out
    finally:
        _ok(hip.hipGraphDestroy(graph))
