import ctypes
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as orc
    orc.build()
    return orc


class _KernelNodeParams(ctypes.Structure):      # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


@pytest.fixture(scope="session")
def kernels_of():
    """kernels_of(call): the kernels that `call` launches, as (name, grid) in order.  The call is recorded into a graph
    that is never run, so its tensors may be stand-ins."""
    import torch
    with open("/proc/self/maps") as maps:      # the runtime that is loaded, not another copy of it
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p

    def kernels(call):
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g):
            call()
        graph, n = ctypes.c_void_p(g.raw_cuda_graph()), ctypes.c_size_t(0)
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        found = []
        for node in nodes:
            kind, p = ctypes.c_int(-1), _KernelNodeParams()
            assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
            assert kind.value == 0, "not a kernel node"
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), None) or b""
            found.append((name.decode(), tuple(p.grid)))
        return found
    return kernels
