"""Prefill attention of many short items, whose workgroups of four wavefronts share a compute unit: edges of their tiles (32 positions of
four heads, 16 of eight, 64 of two, 128 of one), idle wavefronts, and key tiles around the five after which its LDS stages repeat."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu

ROWS = [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 0, 48]
CASES = [   # heads, kv heads, rows, pages
    (8, 2, ROWS * 13, [0, 1, 3, 4, 5, 8, 12, 20, 24, 28, 2, 40] * 13),    # 32 rows and fewer on average: behind any number of keys
    (8, 2, [33, 64, 65, 97] * 36, [0, 2, 7, 17] * 36),
    (8, 1, ROWS[:7] * 40, [0, 4, 16, 23, 24, 25, 33] * 40),               # eight heads
    (16, 1, [17, 33, 5] * 45, [0, 3, 9] * 45),
    (4, 2, [63, 64, 65, 5] * 34, [1, 0, 3, 11] * 34), (3, 1, [127, 128, 129, 40] * 24, [0, 1, 5, 9] * 24), (6, 2, [50, 131] * 25, [2, 8] * 25),
]


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_short_items(case, static):
    from paper_2508_08438_amd import binding as skv
    hq, hkv, S, k = CASES[case]
    c = attn_case(300 + case, len(S), hq, hkv, 128, torch.bfloat16, max(k), S, k, n_pages=sum(k) + 3)
    if static:
        x = {n: (v if torch.is_tensor(v) else torch.from_numpy(v)).to("cuda:0") for n, v in c.items()}
        out = torch.full_like(x["q"], 7.0)
        skv.skv_prefill_attn_static(skv.attn_desc(hq, hkv, 128, "bf16"), x["q"], x["knew"], x["vnew"], x["q_off"], x["kpool"],
                                    x["vpool"], x["matched_len"], x["page_table"], max(k), out)
        got = out.double().cpu().numpy()
    else:
        got = run_attn(c)
    want = oracle.attention(**c, n_threads=16)
    assert np.isfinite(got).all()
    # values to 4.9: the rounding of the weights to 8 bits moves a mean of them by up to 2^-9 of that, the rounding of the output as much again
    assert np.abs(got - want).max() <= 2e-2
