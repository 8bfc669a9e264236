"""cs_bundle_update_launches is the number of launches that the update makes: the kernel nodes of its captured graph."""
import ctypes

import pytest
import torch

import paper_1903_04488_amd as cs
from paper_1903_04488_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RELAXED, KERNEL_NODE = 2, 0                               # hipStreamCaptureModeRelaxed, hipGraphNodeTypeKernel


def _captured_kernels(fn):
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream(DEV)
    stream.wait_stream(torch.cuda.current_stream(DEV))
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize(DEV)
    with torch.cuda.stream(stream):
        handle = ctypes.c_void_p(stream.cuda_stream)
        assert hip.hipStreamBeginCapture(handle, RELAXED) == 0
        try:
            fn()
        finally:
            ended = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
    assert ended == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    kinds = []
    for node in nodes[:n.value]:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        kinds.append(kind.value)
    assert hip.hipGraphDestroy(graph) == 0
    assert set(kinds) <= {KERNEL_NODE}
    return len(kinds)


# one group, a single vector, groups that share a launch with their rest and without, more than a launch takes, rows by list and
# by walk, rows of both kinds, more rows than a launch takes, no lists
@pytest.mark.parametrize("r,c,d,flags", [
    (5, 1 << 15, 1 << 20, 0), (15, 1 << 12, 3_000_000, 0), (15, 1 << 18, 5_000_000, 0), (3, 1 << 16, 9_000_000, 0),
    (5, 70_001, 2_300_001, 0), (7, 100_003, 1_700_001, 0), (5, 1 << 15, 1 << 20, B.CS_FLAG_NO_VISIT_LIST),
    (5, 70_001, 2_300_001, B.CS_FLAG_NO_VISIT_LIST), (5, 1000, 3000, 0)])
def test_launches_of_the_update(r, c, d, flags):
    p = cs.cs_params_init(r, c, 190304488, d)
    p.flags = flags
    g = torch.zeros(d, device=DEV)
    T = torch.zeros(cs.cs_bundle_floats(p, 300), device=DEV)
    for W in (1, 2, 8, 9, 14, 33, 65, 250, 300):
        part = T[:cs.cs_bundle_floats(p, W)]
        made = _captured_kernels(lambda: cs.cs_sketch_accumulate_bundle(p, part, [g] * W))   # noqa: B023
        assert made == cs.cs_bundle_update_launches(p, W, d), W
