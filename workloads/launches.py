"""Which kernels a call launches: the call is captured into a HIP graph and the graph's nodes are read."""
import ctypes
import re

import torch


class _KernelParams(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


def _libraries():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip, cxx = ctypes.CDLL(path), ctypes.CDLL("libstdc++.so.6")
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    cxx.__cxa_demangle.restype = ctypes.c_char_p
    return hip, cxx


def _nodes(call):
    """(kernel with its template arguments, workgroups, threads, function) of the launches of one call, in their order."""
    hip, cxx = _libraries()
    call()                                                    # (workspace and first-launch work outside the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    handle, count = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(count)) == 0
    out = []
    for node in nodes:
        kind, params = ctypes.c_int(), _KernelParams()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0, "not a kernel"
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(params)) == 0
        name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(params.func), None)
        name = cxx.__cxa_demangle(name, None, None, None).decode()
        name = re.sub(r"\(anonymous namespace\)::|comet_gemm::|^void ", "", name)
        out.append((re.sub(r"\((GemmParams|GemmGroup|comet|unsigned|int|void).*", "", name),
                    params.grid[0] * params.grid[1] * params.grid[2], params.block[0], params.func))
    return out


def kernels(call):
    """The names of the kernels that one call launches, in the order of the launches."""
    return [node[0] for node in _nodes(call)]


def places(call, kernel):
    """Workgroups of the launch whose kernel's name begins with ``kernel``, and how many share a compute unit by the
    kernel's registers and LDS."""
    hip, _ = _libraries()
    found = [(grid, threads, func) for name, grid, threads, func in _nodes(call) if name.startswith(kernel)]
    assert len(found) == 1
    grid, threads, func = found[0]
    count = ctypes.c_int(0)
    assert hip.hipOccupancyMaxActiveBlocksPerMultiprocessor(ctypes.byref(count), ctypes.c_void_p(func), threads, ctypes.c_size_t(0)) == 0
    return grid, count.value
