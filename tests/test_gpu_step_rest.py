"""The rest of a bf16 step behind the attention's workgroups, in every form that carries it: every output the same as that of the three
stages, which run the attention without; on both sides of the number of workgroups up to which it does."""
import ctypes

import pytest
import torch

from paper_2508_08438_amd import binding as skv
from test_gpu_step_call import _buffers, _same, _stages, _step

pytestmark = pytest.mark.gpu

CASES = [
    # (query heads, kv heads, rows, blocks): whole items found in place; from a list; whose longest part is long, split from the list
    (8, 8, [64, 20, 0, 33] * 6, [0, 1, 2, 0] * 6), (32, 8, [100, 300, 0, 129, 64] * 4, [30, 1, 40, 0, 7] * 4), (16, 8, [770, 765, 770], [480, 470, 481]),
    # four wavefronts to a workgroup: 100 requests of up to 17 rows (2024 workgroups), 110
    (32, 8, [17, 16, 9, 17] * 25, [2, 0, 3, 1] * 25), (32, 8, [17, 16] * 55, [2, 3] * 55),
    # eight heads and 32-row tiles; a head alone
    (64, 8, [40, 9, 33, 70] * 8, [10, 40, 3, 0] * 8), (3, 3, [130, 300, 5] * 9, [9, 0, 30] * 9),
    # split in place: long parts, the last request without rows; long items that stay whole, the shortest such table and a shorter one
    (32, 8, [900, 0], [1190, 70]), (64, 8, [118] * 4, [180, 0, 177, 180]), (64, 8, [118] * 4, [71] * 4), (64, 8, [118] * 4, [67, 67, 0, 67]),
    # 512 requests, 513
    (4, 1, [5, 0, 33, 2] * 128, [1, 0, 2, 1] * 128), (4, 1, [5, 0, 33] * 171, [1, 0, 2] * 171),
]


class _Node(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def launches(call):
    """Workgroups of each kernel that a call enqueues."""
    call()
    torch.cuda.synchronize()
    g, n, lib = torch.cuda.CUDAGraph(keep_graph=True), ctypes.c_size_t(), skv.lib()
    with torch.cuda.graph(g):
        call()
    graph = ctypes.c_void_p(g.raw_cuda_graph())
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes, p = (ctypes.c_void_p * n.value)(), _Node()
    assert lib.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    grids = []
    for node in nodes:
        assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        grids.append(p.grid[0])
    return grids


@pytest.mark.parametrize("case", range(len(CASES)))
def test_step_is_its_stages(case):
    hq, hkv, S, k = CASES[case]
    desc, c, ws, outputs = _buffers(case + 70, S, k, hq, hkv, 128, "bf16", max(k) + 1)
    want, got = outputs(), outputs()
    ws.fill_(0x5a)
    _stages(desc, c, ws, want)
    ws.fill_(0xa5)
    _step(desc, c, ws, got)
    _same(want, got)


# Either side of the lines of the rule that says so (rest_rides and rides_with_parts of skv_attn.hip).  Behind a list: two kernels, or the copy's in front; a plan
# with parts has two anyway, the attention (a round of 256 workgroups) and the merge, and the copy with one of them.
@pytest.mark.parametrize("hq,hkv,n,rows,blocks,parts,rides", [
    # four wavefronts to a workgroup: 12 MB a pool, 128 rows, any size of page
    (32, 8, 63, 3, 7, False, False), (32, 8, 63, 3, 6, False, True), (32, 8, 20, 128, 20, False, False), (32, 8, 20, 129, 20, False, True),
    (16, 2, 205, 2, 8, False, False), (16, 2, 205, 2, 7, False, True),
    # eight: 16 MB of pages below 16 KB, 128 rows; pages of 32 KB
    (16, 1, 121, 2, 34, False, False), (16, 1, 121, 2, 33, False, True), (16, 1, 20, 128, 210, False, False), (16, 1, 20, 129, 210, False, True),
    (32, 8, 14, 100, 100, False, True),
    # long items that stay whole: 40 key tiles, 39; parts of 125 key tiles
    (64, 8, 4, 118, 148, True, True), (64, 8, 4, 118, 147, True, False), (32, 8, 1, 900, 1190, True, True)])
def test_which_copies_ride(hq, hkv, n, rows, blocks, parts, rides):
    desc, c, ws, outputs = _buffers(n, [rows] * n, [blocks] * n, hq, hkv, 128, "bf16", blocks + 1)
    o = outputs()
    grids = launches(lambda: _step(desc, c, ws, o))
    if parts:
        assert len(grids) == 2 and (grids[0] > 256) == rides, grids
    else:
        assert len(grids) == (2 if rides else 3), grids
