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


def step_kernels(layers, B, mode="auto"):
    """kernel_nodes of one ff_train_step of a stack, over random weights and inputs."""
    from paper_2506_22771_amd import schedule
    g = torch.Generator(device="cuda").manual_seed(3)
    w = [torch.rand((l.N, l.K), generator=g, device="cuda") * 0.4 - 0.2 for l in layers]
    x = [torch.randn((B, layers[0].in_elems_per_sample), generator=g, device="cuda") for _ in range(2)]
    st = schedule.TrainState.from_weights(layers, B, w)
    net = ff.Net(layers, B, st.w_master, st.w_q, st.s_w, launch_mode=mode)
    loss, good = torch.empty((len(layers), 2), device="cuda"), torch.empty((len(layers), 2, B), device="cuda")
    ws = torch.empty(net.workspace_bytes(), dtype=torch.uint8, device="cuda")

    def step():
        ff.ff_train_step(net, x[0], x[1], 2.0, 0.05, 1e-4, 5, 0, loss, good, ws)

    step()
    torch.cuda.synchronize()
    return kernel_nodes(step)
