"""Which kernels a call launches: the call is recorded into a HIP graph, which
is read node by node and never run."""
import ctypes
import re

import torch


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def _hip():
    with open("/proc/self/maps") as f:  # the runtime that is loaded
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    lib = ctypes.CDLL(path)
    lib.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    return lib


def launches(call):
    """[(mangled kernel name, workgroups, threads per workgroup)] of
    call(stream), in the order of their recording."""
    hip, p = _hip(), ctypes.c_void_p

    def check(rc, what):
        assert rc == 0, f"{what}: HIP error {rc}"

    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph, st = p(), p(stream.cuda_stream)
    check(hip.hipStreamBeginCapture(st, 2), "hipStreamBeginCapture")  # relaxed
    try:
        call(stream)
    finally:
        check(hip.hipStreamEndCapture(st, ctypes.byref(graph)), "hipStreamEndCapture")
    n = ctypes.c_size_t()
    check(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)), "hipGraphGetNodes")
    nodes = (p * n.value)()
    check(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)), "hipGraphGetNodes")
    found = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        check(hip.hipGraphNodeGetType(p(node), ctypes.byref(kind)), "hipGraphNodeGetType")
        assert kind.value == 0, f"node of type {kind.value}, not a kernel"
        k = _KernelNodeParams()
        check(hip.hipGraphKernelNodeGetParams(p(node), ctypes.byref(k)), "hipGraphKernelNodeGetParams")
        found.append((hip.hipKernelNameRefByPtr(p(k.func), st).decode(), k.grid.x * k.grid.y * k.grid.z,
                      k.block.x * k.block.y * k.block.z))
    check(hip.hipGraphDestroy(graph), "hipGraphDestroy")
    return found


def kernels(call):
    """Kernel names with the values of their template arguments, as 'k_name<1,0>'
    (without them where an argument is a type)."""
    out = []
    for name, _, _ in launches(call):
        m = re.match(r"_ZN3spk(\d+)", name)
        assert m, name
        base, rest = name[m.end():][:int(m[1])], name[m.end() + int(m[1]):]
        args = re.match(r"I((?:L[a-z]n?\d+E)+)E", rest)
        out.append(base + (f"<{','.join(re.findall(r'L[a-z](n?[0-9]+)E', args[1]))}>" if args else ""))
    return out
