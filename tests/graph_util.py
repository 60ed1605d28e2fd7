"""Which kernels a call launches and what each waits for, read off the graph it is captured into.  Nothing is replayed."""
import ctypes as C

import torch

import paper_2506_22771_amd as ff


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNodeParams(C.Structure):
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p),
                ("shared", C.c_uint)]


def kernel_nodes(call):
    """(kernel name, names of the kernels it waits for) of every kernel that `call` launches.  Streams of the library have to exist
    before: run the call once."""
    hip = ff.lib()   # (symbols of the runtime it is linked to)
    hip.hipKernelNameRefByPtr.restype = C.c_char_p
    cuda_graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(cuda_graph):
        call()
    graph = C.c_void_p(cuda_graph.raw_cuda_graph())

    def ok(status):
        assert status == 0, status

    def name(node):
        kind = C.c_int(-1)
        ok(hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)))
        if kind.value != 0:   # hipGraphNodeTypeKernel
            return ""
        p = _KernelNodeParams()
        ok(hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)))
        return hip.hipKernelNameRefByPtr(C.c_void_p(p.func), None).decode()

    n = C.c_size_t(0)
    ok(hip.hipGraphGetNodes(graph, None, C.byref(n)))
    nodes = (C.c_void_p * max(1, n.value))()
    if n.value:
        ok(hip.hipGraphGetNodes(graph, nodes, C.byref(n)))
    out = []
    for node in nodes[:n.value]:
        m = C.c_size_t(0)
        ok(hip.hipGraphNodeGetDependencies(C.c_void_p(node), None, C.byref(m)))
        deps = (C.c_void_p * max(1, m.value))()
        if m.value:
            ok(hip.hipGraphNodeGetDependencies(C.c_void_p(node), deps, C.byref(m)))
        out.append((name(node), [name(d) for d in deps[:m.value]]))
    return [e for e in out if e[0]]
