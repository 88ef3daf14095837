"""bf16 prefill attention where workgroups find their items themselves (up to 64 requests) and where a list is made in front: on both
sides of every limit between them, with and without items split along the keys.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu

PLAN = [
    # (query heads, kv heads, suffix rows, cached blocks): one item; no rows; 30, 32, 33 requests of a split call (62 .. 66 items at most);
    (8, 8, [1], [0]), (8, 8, [0, 0], [3, 0]), (8, 8, [0, 7, 0], [3, 40, 0]),
    (8, 1, [1] * 30, [60] * 30), (8, 1, [1] * 32, [60] * 32), (8, 1, [1] * 33, [60] * 33), (8, 1, [2] * 70, [70] * 70),
    # short first tiles and tiles cut from row 0; heads alone, in pairs, four and eight; lengths far apart
    (4, 4, [300, 5], [90, 300]), (4, 2, [200, 1, 0, 129], [33, 250, 4, 100]), (32, 8, [137], [187]), (64, 8, [257, 3], [500, 7]),
    (16, 2, [64, 65, 63, 1], [4, 9, 130, 260]),
    # unsplit: 63, 64, 65 requests; eight rounds of workgroups and more, from a list
    (8, 2, [33, 70] * 31 + [1], [1, 9] * 31 + [80]), (8, 2, [33, 70] * 32, [1, 9] * 32), (8, 2, [33, 70] * 32 + [1], [1, 9] * 32 + [80]),
    (32, 8, [65] * 60 + [900], [2] * 61), (32, 8, [200] * 64, [2] * 64), (32, 8, [260] * 64, [0, 1] * 32),
]


@pytest.mark.parametrize("case", range(len(PLAN)))
def test_items(case):
    hq, hkv, S, k = PLAN[case]
    c = attn_case(300 + case, len(S), hq, hkv, 128, torch.bfloat16, max(k) + 1, S, k, n_pages=sum(k) + 3)
    r = int(np.argmax(k))
    if k[r] > 3:                      # an absent page reads as zeros
        for pool in ("kpool", "vpool"):
            c[pool][c["page_table"][r, 2]] = 0
    want = oracle.attention(**c, n_threads=16)
    if k[r] > 3:
        c["page_table"][r, 2] = -1 if case % 2 else sum(k) + 9
    got = run_attn(c)
    assert got.shape == want.shape and np.isfinite(got).all()
    assert got.size == 0 or np.abs(got - want).max() <= 2e-2
