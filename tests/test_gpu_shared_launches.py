"""How many launches uniql_w4_linear_multi makes of a set of linears, counted as nodes of a captured graph: the members that one
kernel takes share one; and the same bits as separate calls, on first launch and on replay."""
import ctypes as C

import numpy as np
import pytest

import workloads as wl
from workloads import Keep

pytestmark = pytest.mark.gpu


def nodes(torch, graph):
    hip = C.CDLL("libamdhip64.so")
    n = C.c_size_t(0)
    hip.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    assert hip.hipGraphGetNodes(graph.raw_cuda_graph(), None, C.byref(n)) == 0
    return n.value


SEG = Keep(k_keep=8 * 108, col_seg_stride=128, col_seg_keep=108)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M,specs,launches", [
    (8, [(6500, 1024, Keep()), (200, 1024, Keep()), (129, 1024, Keep())], 1),          # a decode batch, tall and short
    (12, [(6500, 1024, Keep()), (200, 1024, Keep()), (129, 1024, Keep())], 1),
    (12, [(6500, 2304, Keep()), (200, 1024, Keep()), (129, 1024, Keep())], 1),         # (rows of different lengths)
    (12, [(6500, 4224, Keep()), (200, 1024, Keep()), (129, 1024, Keep())], 2),         # the tall one, whose rows are long, by itself
    (24, [(6500, 1152, Keep()), (200, 1024, Keep()), (6401, 1024, Keep(k_keep=1001)), (48, 1024, Keep())], 1),
    (24, [(6500, 4352, Keep()), (200, 1024, Keep()), (6401, 4224, Keep(k_keep=4201)), (48, 1024, Keep())], 2),   # two and two
    (12, [(200, 1024, SEG), (129, 1024, Keep()), (97, 1152, Keep(k_keep=1100))], 2),   # segments do not share a decode batch
    (40, [(6500, 1024, Keep()), (200, 1024, Keep()), (129, 1024, Keep())], 2),         # two ways to split K
    (40, [(200, 1024, Keep()), (129, 1024, Keep())], 1),
    (40, [(200, 1024, SEG), (129, 1024, Keep()), (97, 1024, SEG), (65, 1152, Keep())], 2),
    (40, [(200, 896, Keep()), (129, 1024, Keep()), (97, 896, Keep())], 3),             # short rows do not share
    (100, [(200, 1024, Keep()), (129, 1152, Keep()), (97, 1024, Keep())], 1),
])
def test_launches_and_bits(M, specs, launches, fmt):
    import torch
    import paper_2512_03383_amd as uq
    rng = wl.rng_for(72, M)
    tdt = torch.bfloat16 if fmt == "bf16" else torch.float16
    ws = [uq.QuantLinear.from_numpy(wl.gen_linear(rng, N, K, fmt=fmt)) for N, K, _ in specs]
    keeps = [k for _, _, k in specs]
    dims = [uq.kept_dims(w, k) for w, k in zip(ws, keeps)]
    xs = [torch.randn((M, kk), device="cuda").to(tdt) for _, kk in dims]
    ys = [torch.empty((M, nk), dtype=tdt, device="cuda") for nk, _ in dims]
    want = [uq.uniql_w4_linear(w, k, x) for w, k, x in zip(ws, keeps, xs)]
    call = uq.MultiCall(ws, keeps, xs, ys)
    call.run()
    torch.cuda.synchronize()
    assert all(torch.equal(y, t) for y, t in zip(ys, want))
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call.run()
    assert nodes(torch, graph) == launches
    graph.instantiate()
    for _ in range(3):
        for y in ys:
            y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(y, t) for y, t in zip(ys, want))
