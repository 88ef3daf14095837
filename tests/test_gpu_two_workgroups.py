"""Prefill attention of many short items, whose workgroups of four wavefronts share a compute unit: edges of their tiles (32 positions of
four heads, 16 of eight, 64 of two, 128 of one), idle wavefronts, and key tiles around the five after which its LDS stages repeat."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_beside import _results, _ruin, _session
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


def _items(S, k, rows):
    """q tiles of the requests: the first one is short where the cached keys end inside a key tile, unless that costs a tile."""
    n = 0
    for s, L in zip(S, 16 * np.asarray(k)):
        head = min(s, -L & min(63, rows - 1))
        tiles, plain = (head > 0) + -(-(s - head) // rows), -(-s // rows)
        n += plain if plain < tiles and 2 * L > s else tiles
    return n


def _run(c, nbytes=None):
    """The output, and the items listed."""
    from paper_2508_08438_amd import binding as skv
    x = {n: (v if torch.is_tensor(v) else torch.from_numpy(v)).to("cuda:0") for n, v in c.items()}
    desc = skv.attn_desc(x["q"].shape[1], x["kpool"].shape[2], 128, "bf16")
    full = skv.skv_prefill_attn_workspace_size(desc, len(x["matched_len"]), len(x["q"]))
    ws, out = torch.zeros(nbytes or full, dtype=torch.uint8, device="cuda:0"), torch.full_like(x["q"], 7.0)
    skv.skv_prefill_attn(desc, x["q"], x["knew"], x["vnew"], x["q_off"], x["kpool"], x["vpool"], x["matched_len"], x["page_table"],
                         x["page_table"].shape[1], out, ws)
    torch.cuda.synchronize()
    return out.cpu(), int(ws[:4].view(torch.int32))


@pytest.mark.parametrize("values", ["plain", "wide", "weightless", "absent"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_values_and_the_larger_form(case, values):
    """Scores that spread over a hundred and move the softmax reference, scores of -infinity in front, absent pages: against the oracle, and
    bit for bit the form of eight wavefronts, which a workspace too small for the longer list gets."""
    hq, hkv, S, k = CASES[case]
    c = attn_case(400 + case, len(S), hq, hkv, 128, torch.bfloat16, max(k), S, k, n_pages=sum(k) + 3)
    if values == "wide":
        c["q"] *= 16
    if values == "weightless":
        c["q"] = c["q"].abs() + 0.01
        for r in range(0, len(S), 3):
            for j in range(k[r] * 2 // 3):
                c["kpool"][c["page_table"][r, j]] = float("-inf")
    gone = [(r, (7 * r) % k[r]) for r in range(0, len(S), 2) if k[r]] if values == "absent" else []
    for r, j in gone:                  # read as zeros
        for pool in ("kpool", "vpool"):
            c[pool][c["page_table"][r, j]] = 0
    want = oracle.attention(**c, n_threads=16)
    for i, (r, j) in enumerate(gone):
        c["page_table"][r, j] = -1 if i % 2 else sum(k) + 9
    got, items = _run(c)
    G, pad = hq // hkv, lambda n: (n + 255) // 256 * 256
    heads = 8 if G % 8 == 0 else 4 if G % 4 == 0 else 2 if G % 2 == 0 else 1
    assert items == _items(S, k, 128 // heads)
    # the weights, of which few count where scores are wide, and the output are rounded to 8 bits: by up to 2^-8 of each
    vmax = float(max(c["vpool"].abs().max(), c["vnew"].abs().max()))
    assert np.isfinite(want).all() and (np.abs(got.double().numpy() - want) <= 2.0 ** -8 * (vmax + np.abs(want)) + 1e-5).all()
    rows = 256 // min(heads, 4)
    other, items = _run(c, 256 + pad(4096 * hkv) + pad(32 * (sum(S) // rows + 2 * len(S))))
    assert items == _items(S, k, rows) and torch.equal(got, other)


def test_copy_beside(monkeypatch):
    s = _session(monkeypatch, 500, 1 << 60)
    _ruin(s)
    s.step()
    want = _results(s)
    s = _session(monkeypatch, 500, 0)
    for _ in range(4):
        _ruin(s)
        s.step()
        assert all(torch.equal(a, b) for a, b in zip(want.values(), _results(s).values()))
    S, k = np.diff(want["q_off"].numpy()), want["matched_len"].numpy() // 16
    assert int(s.workspace[:4].view(torch.int32)) == _items(S, k, 32) > 256
