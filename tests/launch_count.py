"""Number of kernels a call launches: it is captured into a HIP graph, whose nodes are counted."""
import ctypes

import torch

HIP_NODE_KERNEL = 0


class KernelNode(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def kernel_launches(call, stream):
    """Kernel nodes of `call` (which enqueues work on `stream` only), captured and thrown away."""
    return len(kernel_nodes(call, stream))


def kernel_nodes(call, stream):
    """Block, grid and dynamic LDS of the kernels `call` launches on `stream`."""
    hip = ctypes.CDLL("libamdhip64.so")
    s, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()

    def ok(rc):
        assert rc == 0, rc

    torch.cuda.synchronize()
    ok(hip.hipStreamBeginCapture(s, 2))                     # relaxed
    try:
        call()
    finally:
        ok(hip.hipStreamEndCapture(s, ctypes.byref(graph)))
    ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
    nodes = (ctypes.c_void_p * n.value)()
    ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
    kernels = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        ok(hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)))
        if kind.value == HIP_NODE_KERNEL:
            kernels.append(KernelNode())
            ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(kernels[-1])))
    ok(hip.hipGraphDestroy(graph))
    return kernels
