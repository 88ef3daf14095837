"""Split calls whose parts are shorter in two rounds of workgroups, and neighbours of theirs that stay in one.  Against the fp64 oracle; the
work list's count, which the workspace begins with, says that more parts were dealt than one round holds (0: no list was made)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08438_amd import binding as skv
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu


# query heads over one kv head, rows, blocks, parts.  An item is 64 rows and 3, 5 or 7 workgroups: rounds hold 85, 51 and 36
@pytest.mark.parametrize("hq,rows,blocks,parts", [
    (28, 65, [427, 213, 213, 213, 427, 341, 213, 427, 128, 213], 72),
    (20, 130, [110, 367, 110, 183, 183, 367, 183, 110, 110, 183], 96),
    (12, 200, [117, 117, 393, 393, 196, 393, 393, 117, 196, 117, 393], 166),
    # as many items as leave nothing to split in one round, of lengths that do not say so: 150 key tiles and 148
    (28, 129, [600, 150, 600, 150, 600, 150, 600, 150, 600], 72), (28, 129, [580, 150, 580, 150, 580, 150, 580, 150, 580], 0),
    # a quarter of the keys; one request of them
    (28, 65, [106, 53, 53, 53, 106, 85, 53, 106, 32, 53], 0), (28, 65, [427], 0), (12, 200, [393, 117], 0),
])
def test_rounds(monkeypatch, hq, rows, blocks, parts):
    n = len(blocks)
    c = attn_case(n + hq, n, hq, 1, 128, torch.bfloat16, max(blocks) + 1, [rows] * n, blocks, n_pages=sum(blocks) + 3)
    seen = []
    call = skv.skv_prefill_attn
    monkeypatch.setattr(skv, "skv_prefill_attn", lambda *a: (seen.append(a[-1]), call(*a)))
    got, want = run_attn(c), oracle.attention(**c, n_threads=16)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= 2e-2
    assert int(seen[0][:4].view(torch.int32)) == parts
