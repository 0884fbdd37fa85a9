"""The kernel launches of a call, read from a graph it is captured into: which route a dispatch took shows in their number, grids
and workgroup sizes."""
import ctypes as C

import torch


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


class _KernelParams(C.Structure):
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p),
                ("lds", C.c_uint)]


def _hip():
    with open("/proc/self/maps") as f:
        path = next(ln.split()[-1] for ln in f if "libamdhip64.so" in ln)
    lib = C.CDLL(path)
    lib.hipGraphGetNodes.argtypes = [C.c_void_p, C.POINTER(C.c_void_p), C.POINTER(C.c_size_t)]
    lib.hipGraphNodeGetType.argtypes = [C.c_void_p, C.POINTER(C.c_int)]
    lib.hipGraphKernelNodeGetParams.argtypes = [C.c_void_p, C.POINTER(_KernelParams)]
    return lib


def _kernels(call):
    hip = _hip()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    raw, count = graph.raw_cuda_graph(), C.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, C.byref(count)) == 0
    nodes = (C.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(count)) == 0
    for node in nodes:
        kind, p = C.c_int(-1), _KernelParams()
        assert hip.hipGraphNodeGetType(node, C.byref(kind)) == 0 and kind.value == 0, "not a kernel launch"
        assert hip.hipGraphKernelNodeGetParams(node, C.byref(p)) == 0
        yield p


def of(call):
    """[(workgroups, threads of a workgroup, bytes of dynamic LDS)] in the order of the graph's nodes (captured, not run)."""
    return [(p.grid.x * p.grid.y * p.grid.z, p.block.x * p.block.y * p.block.z, p.lds) for p in _kernels(call)]


def functions(call):
    """The kernels themselves, as numbers that are equal where two launches run the same one."""
    return [p.func for p in _kernels(call)]


def named(call, kernel):
    """(name, addresses of its arguments) of every launch of a kernel with `kernel` in its name, while its graph is there."""
    hip = _hip()
    hip.hipKernelNameRefByPtr.restype, hip.hipKernelNameRefByPtr.argtypes = C.c_char_p, [C.c_void_p, C.c_void_p]
    for p in _kernels(call):
        name = hip.hipKernelNameRefByPtr(p.func, None).decode()
        if kernel in name:
            yield name, C.cast(p.params, C.POINTER(C.c_void_p))


def words(address, n):
    """n 32-bit integers from there (no more than the argument has)."""
    return list((C.c_int32 * n).from_address(address))
