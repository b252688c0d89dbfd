"""homs_batched_config.grid is the number of workgroups of the persistent kernel
for every engine, as the header says: read from the launches of a captured
search, whose results do not depend on it."""
import ctypes

import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X GPU")]

from synth import WORKLOADS, make_workload  # noqa: E402


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNode(ctypes.Structure):
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", _Dim3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _launches(hip, stream, call):
    """(grid, block) of every kernel that `call` launches on the stream"""
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream), 1) == 0  # thread-local
    call()
    assert hip.hipStreamEndCapture(ctypes.c_void_p(stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p, kind = _KernelNode(), ctypes.c_int()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value == 0:  # a kernel
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            out.append((p.grid.x, p.block.x))
    assert hip.hipGraphDestroy(graph) == 0
    return out


@pytest.mark.parametrize("grid", [1, 100, 777, 2048])
def test_grid_is_the_number_of_workgroups(grid):
    import torch
    import paper_2211_16422_amd.hyperoms as h

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")

    hip = ctypes.CDLL(h.LIB_PATH)  # the runtime it is linked with
    g = make_workload(WORKLOADS["tiny"], n_ref=3000, n_query=600, seed=5)
    lib, q = g.library, g.queries
    hp = h.Params(dim=1024)
    with h.Context(hp) as ctx:
        ctx.encode_library(*h.to_device_csr(*h.preprocess(hp, lib.offsets, lib.mz, lib.intensity),
                                            "cuda:0"), dev(lib.pmz), dev(lib.charge))
        hv = ctx.encode_queries(*h.to_device_csr(*h.preprocess(hp, q.offsets, q.mz, q.intensity),
                                                 "cuda:0"))
        kinds = dev((np.arange(q.n) % 2).astype(np.int8))
        values = dev(np.where(np.arange(q.n) % 2, 20.0, 500.0))
        args = (hv, dev(q.pmz), dev(q.charge), kinds, values)
        default = ctx.batched_config()
        want = ctx.search_batched(*args, use_graph=False)
        for engine, threads in ((h.ENGINE_POPCOUNT, 256), (h.ENGINE_MFMA_F8, 512),
                                (h.ENGINE_MFMA_F4, 512)):
            ctx.set_batched_config(**dict(default, engine=engine, grid=grid, narrow_max=16))
            got = ctx.search_batched(*args, use_graph=False)  # and the workspace is there
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), engine
            idx, dist = torch.empty_like(want[0]), torch.empty_like(want[1])
            s = torch.cuda.Stream()
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                launches = _launches(hip, s.cuda_stream, lambda: ctx.search_batched(
                    *args, use_graph=False, out_idx=idx, out_dist=dist))
            assert (grid, threads) in launches, (engine, launches)
