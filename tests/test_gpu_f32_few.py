"""fp32 prefill attention of few items, whose keys eight wavefronts share (more than 256 of them), is as exact as that of many, where four do: the same requests alone
and in enough copies, both against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu


def _copies(c, n):
    R, T = len(c["matched_len"]), len(c["q"])
    off = np.concatenate([c["q_off"][:-1] + i * T for i in range(n)] + [[n * T]]).astype(np.int32)
    rep = lambda x: x.repeat(n, *[1] * (x.dim() - 1))
    return dict(c, q=rep(c["q"]), knew=rep(c["knew"]), vnew=rep(c["vnew"]), q_off=off, matched_len=np.tile(c["matched_len"], n),
                page_table=np.tile(c["page_table"], (n, 1)))


# (rows / 32 + requests) * heads items: up to 256 alone, more than 256 and fewer than 1024 in copies.  Both are of the same precision, so the
# mean over the shapes is compared: a single one differs by up to 1 % either way
def test_few_items_are_as_exact():
    ratio = []
    for hq, hkv, S, k, n in [(8, 8, [64], [16], 16), (8, 2, [100, 37], [40, 21], 6), (4, 2, [300], [12], 8), (8, 8, [132], [56], 7), (4, 4, [33] * 3, [90] * 3, 14),
                             (8, 4, [97], [20], 9), (16, 4, [60, 20], [30, 75], 5)]:
        c = attn_case(hq + sum(S), len(S), hq, hkv, 64, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
        items = lambda m: (m * sum(S) // 32 + m * len(S)) * hq
        assert items(1) <= 256 < items(n) < 1024
        want = oracle.attention(**c, n_threads=16)
        few, many = run_attn(c), run_attn(_copies(c, n))[: len(want)]
        assert not np.array_equal(few, many)
        ratio.append(np.linalg.norm(few - want) / np.linalg.norm(many - want))
    assert np.mean(ratio) <= 1.0, ratio


# a table of up to 256 keys: four wavefronts here too, hence the same bits; one block or row more: eight
@pytest.mark.parametrize("S,k,eight", [([1], [15], False), ([40, 3], [0, 5], False), ([256], [3], False), ([33] * 9, [15] * 9, False),
                                       ([33] * 9, [16] * 9, True), ([257], [15], True)])
def test_few_keys_take_four_wavefronts(S, k, eight):
    c = attn_case(sum(S), len(S), 8, 8, 64, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    n, items = next((m, i) for m in range(2, 99) if (i := (m * sum(S) // 32 + m * len(S)) * 8) > 256)
    assert (sum(S) // 32 + len(S)) * 8 <= 256 and items < 1024
    few, many = run_attn(c), run_attn(_copies(c, n))[: sum(S)]
    assert np.array_equal(few, many) != eight
    assert np.abs(few - oracle.attention(**c, n_threads=16)).max() <= 1e-5
