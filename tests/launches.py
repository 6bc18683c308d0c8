"""Which kernels a call of the library launches: the call is captured into a HIP graph that is never run, and the graph's kernel
nodes are listed.  For tests whose subject is a kernel that the dispatch takes by itself."""
import ctypes as C
import re


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNodeParams(C.Structure):
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p),
                ("shared", C.c_uint32)]


RELAXED, KERNEL_NODE = 2, 0


def launched_kernels(lib, stream, call):
    """-> [(mangled name, (grid x, y, z), block x)] in launch order.  stream: the torch stream (not the default one) that call()
    launches on; call() must neither wait nor allocate.  The HIP entry points are those the library itself is linked to."""
    def ok(rc):
        assert rc == 0, "HIP error %d" % rc

    lib.hipKernelNameRefByPtr.restype = C.c_char_p
    st, graph, n = C.c_void_p(stream.cuda_stream), C.c_void_p(), C.c_size_t(0)
    ok(lib.hipStreamBeginCapture(st, C.c_int(RELAXED)))
    try:
        call()
    finally:
        rc = lib.hipStreamEndCapture(st, C.byref(graph))
    ok(rc)
    ok(lib.hipGraphGetNodes(graph, None, C.byref(n)))
    nodes = (C.c_void_p * n.value)()
    ok(lib.hipGraphGetNodes(graph, nodes, C.byref(n)))
    out = []
    for node in nodes:
        kind, p = C.c_int(-1), _KernelNodeParams()
        ok(lib.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)))
        if kind.value != KERNEL_NODE:
            continue
        ok(lib.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)))
        name = lib.hipKernelNameRefByPtr(C.c_void_p(p.func), st)
        out.append(((name or b"").decode(), (p.grid.x, p.grid.y, p.grid.z), p.block.x))
    ok(lib.hipGraphDestroy(graph))
    return out


def template_ints(name):
    """The integer (and truth value) template arguments of a mangled kernel name, in order."""
    return [int(x) for x in re.findall(r"L[ib](\d+)E", name)]
