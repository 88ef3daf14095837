"""fp32 prefill attention in tiles of 128 rows (which calls: in_tiles below): tiles dealt out by their number among
64 requests at a time, a first tile of what a request's rows leave over, blocks of 32 keys two at a time, a reference that moves when weights
grow.  Against the fp64 oracle; bound as in test_gpu_f32_precision.py."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu
REL = 8 * 2.0 ** -24

G = np.random.default_rng(9)
EDGES = [49, 127, 128, 129, 160, 161, 255, 256, 257, 31, 1, 0, 33, 384, 97, 1100]
# query / kv heads, rows and reused blocks per request
CASES = {
    "edges of tiles": (32, 2, EDGES, [0, 1, 2, 3, 4, 5, 6, 7, 0, 9, 1, 3, 2, 1, 20, 0]),
    "more than 64 requests": (4, 4, G.integers(49, 160, 130), [*G.integers(0, 4, 129), 20]),
    "one of them alone in its 64": (8, 8, [100] * 64 + [130], [1] * 64 + [20]),
    "no rows among them": (16, 4, [0] * 70 + [700] * 11 + [0] * 3, [2] * 75 + [20] + [2] * 8),
    "pages of more than 64 blocks of keys": (64, 4, [200, 330, 100, 164], [260, 129, 128, 0]),
    "one long request": (32, 4, [1500], [5]),
}


def in_tiles(hq, S, max_blocks):
    """Whether such a call is taken in tiles of 128 rows (large_tiles of skv_attn_f32.hip)."""
    T, n = int(sum(S)), len(S)
    rows, items = -(-T // n), (T // 32 + n) * hq
    tiles, keys = -(-rows // 128), max(rows, 16 * max_blocks)
    if T // 128 >= 2 * n and T // 128 * hq >= 512:
        return True
    if items >= 4096 or (items >= 2048 and max_blocks <= 16) or (items >= 1024 and max_blocks <= 2):
        return 100 * rows > 65 * 128 * tiles and keys > 160 + min(n * tiles * hq, 4096) // 20
    return rows >= (64 if 448 < n * tiles * hq <= 512 else 96) * tiles and items >= (1408 if keys > 512 else 1088)


def case(name, seed=3):
    hq, hkv, S, k = CASES[name]
    assert in_tiles(hq, S, max(max(k), 1))
    return attn_case(seed, len(S), hq, hkv, 64, torch.float32, max(max(k), 1), S, k, n_pages=int(sum(k)) + 3)


def check(c, rel=REL):
    want = oracle.attention(**c, n_threads=16)
    got = run_attn(c)
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("error against 64 bits: %.3e" % err)
    assert err <= rel


@pytest.mark.parametrize("name", CASES)
def test_tiles(name):
    check(case(name))


# Scores that grow along the keys: the reference moves in every block, and in some rows only.  Bound: the scores themselves are not small
# here, and one of s (in exp2 units) carries s 2^-24 of its own rounding beside the 8 * 2^-24 of the exponent's argument; the rows' largest
# scores, whose weights count, are `size` on average over rows and heads.
@pytest.mark.parametrize("name", ["edges of tiles", "pages of more than 64 blocks of keys"])
def test_growing_scores(name):
    c = case(name)
    c["kpool"] = c["kpool"].abs()
    c["knew"] = c["knew"].abs()
    c["q"][: len(c["q"]) // 2] = c["q"][: len(c["q"]) // 2].abs() * 2     # (towards larger scores; the others take both signs)
    for r in range(len(c["matched_len"])):
        n = c["q_off"][r + 1] - c["q_off"][r]
        c["knew"][c["q_off"][r]: c["q_off"][r + 1]] *= torch.linspace(0.1, 2.0, int(n) + 1)[1:, None, None]
    G = c["q"].shape[1] // c["knew"].shape[1]
    size = [(c["q"][a:b, h] @ c["knew"][a:b, h // G].T).tril().amax(1).mean() for a, b in zip(c["q_off"][:-1], c["q_off"][1:]) if b > a
            for h in range(c["q"].shape[1])]
    size = float(np.mean(size)) / 8 * 1.4427
    check(c, REL + size * 2.0 ** -24)


def test_absent_pages_read_as_zeros():
    c = case("pages of more than 64 blocks of keys")
    c["page_table"][0, 3] = -1
    c["page_table"][0, 200] = c["kpool"].shape[0]
    c["page_table"][1, 128] = -1
    want_c = dict(c)
    zero = torch.zeros_like(c["kpool"][:1])                               # the oracle reads a page of zeros in their place
    want_c["kpool"], want_c["vpool"] = torch.cat([c["kpool"], zero]), torch.cat([c["vpool"], zero])
    pt = c["page_table"].copy()
    pt[0, 3] = pt[0, 200] = pt[1, 128] = c["kpool"].shape[0]
    want = oracle.attention(**dict(want_c, page_table=pt), n_threads=16)
    got = run_attn(c)
    assert np.linalg.norm(got - want) <= REL * np.linalg.norm(want)


# Either side of the lines of that rule.  The rows of a call that is not in tiles have the bits that they have in a call with single rows
# behind them, which keep the mean below any tile; those of one that is have others.
@pytest.mark.parametrize("hq,n,rows,max_blocks,tiles", [
    (8, 67, 187, 12, False), (8, 67, 187, 14, True), (8, 90, 160, 24, False), (8, 90, 170, 24, True), (32, 290, 150, 11, False),   # alone
    (8, 64, 63, 20, False), (8, 64, 64, 20, True), (8, 65, 95, 20, False), (8, 65, 96, 20, True), (8, 56, 95, 20, False), (8, 57, 95, 20, True), (8, 18, 200, 20, False), (8, 19, 200, 20, True), (8, 19, 200, 33, False),
    (16, 3, 790, 50, False), (16, 4, 790, 50, True),
    (8, 130, 255, 16, False), (8, 130, 256, 16, True)])
def test_which_calls(hq, n, rows, max_blocks, tiles):
    S, more = [rows] * n, n * rows // 40
    assert in_tiles(hq, S, max_blocks) == tiles and not in_tiles(hq, S + [1] * more, max_blocks)
    c = attn_case(rows, n + more, hq, max(hq // 4, 1), 64, torch.float32, max_blocks, S + [1] * more, [min(2, max_blocks)] * (n + more), n_pages=2 * (n + more) + 3)
    T, alone = n * rows, {x: c[x][:n * rows] for x in ("q", "knew", "vnew")}
    got = run_attn(dict(c, **alone, q_off=c["q_off"][:n + 1], matched_len=c["matched_len"][:n], page_table=c["page_table"][:n]))
    assert np.array_equal(got, run_attn(c)[:T]) != tiles


# Nothing behind a request's last key is read: new rows that end where the batch does, in the middle of 16, with NaN behind them.  A NaN
# among the values, its weight 0, would send the tile to the form that takes its rows one by one, whose bits are others.
@pytest.mark.parametrize("n", [1, 4, 5, 8, 11, 15])
def test_nothing_behind_the_last_row(n):
    S, k = [200, 330, 128 + n], [3, 0, 2]
    c = attn_case(n, 3, 64, 4, 64, torch.float32, 3, S, k)
    assert in_tiles(64, S, 3)
    T, got = len(c["knew"]), {}
    for behind in (0.0, float("nan")):
        for x in ("knew", "vnew"):
            full = torch.full((T + 32, *c[x].shape[1:]), behind, device="cuda:0")
            full[:T] = c[x]
            got[x] = full[:T]
        got[str(behind)] = run_attn(dict(c, **{x: got[x] for x in ("knew", "vnew")}))
    assert np.array_equal(got["0.0"], got["nan"])
    want = oracle.attention(**c, n_threads=16)
    assert np.linalg.norm(got["nan"] - want) <= REL * np.linalg.norm(want)
