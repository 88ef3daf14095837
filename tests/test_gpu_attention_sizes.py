"""Prefill attention at the sizes where its kernels change form: edges of row tiles and key blocks, many and empty
requests, absent pages.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu

# fp32: a softmax weight 2^x carries a relative error of about |x| 2^-23 (the rounding of the exponent's argument, |x| <=
# 40 for these scores), the two sums add less; a weighted mean of values up to 5 is then within 5 * 40 * 2^-23 = 2.4e-5.
F32_TOL = 4e-5


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (4, 2, 64), (2, 2, 128), (8, 2, 128)])
@pytest.mark.parametrize("S,k", [
    ([1], [0]), ([1], [1]), ([31, 32, 33, 1], [0, 2, 1, 3]),     # one block of keys, one tile of rows, one more
    ([127, 128, 129, 0, 97], [0, 0, 8, 3, 7]),                   # keys for one round of the four wavefronts, and one more
    ([300], [20]),
    ([0, 0, 3] + [5, 0, 33] * 43 + [0], [1] * 133),              # more than 64 requests, empty ones among them
])
def test_fp32_tiles_and_key_blocks(hq, hkv, d, S, k):
    c = attn_case(sum(S) + hq + d, len(S), hq, hkv, d, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= F32_TOL


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_absent_pages_read_as_zeros(d):
    c = attn_case(5, 3, 4, 2, d, torch.float32, 9, [1, 20, 70], [1, 5, 9], n_pages=40)
    for r, j in ((0, 0), (1, 1), (1, 4), (2, 0), (2, 8)):
        for pool in ("kpool", "vpool"):
            c[pool][c["page_table"][r, j]] = 0
    want = oracle.attention(**c, n_threads=8)
    for n, (r, j) in enumerate(((0, 0), (1, 1), (1, 4), (2, 0), (2, 8))):
        c["page_table"][r, j] = -1 if n % 2 else 40 + n
    assert np.abs(run_attn(c) - want).max() <= F32_TOL


def test_fp32_maxima_that_keep_moving():
    # scores rising over hundreds of exp2 units along the keys: every block moves the running maximum.  The weights that
    # count lie within a few units of the maximum; their score is rounded at 2^-24 * 400, five of those per exponent.
    c = attn_case(9, 2, 2, 2, 64, torch.float32, 5, [200, 90], [4, 0])
    c["q"][:] = 1.0
    n = c["knew"].shape[0]
    c["knew"][:] = torch.arange(n, dtype=torch.float32)[:, None, None] * 0.05
    c["kpool"][:] = -1.0
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.abs(got - want).max() <= 5 * 5 * 400 * 2.0 ** -24


# Long suffixes in number: 128-row tiles of d 64 (32 tiles of 16 heads and more).  Edges of wavefronts, tiles and key tiles.
LARGE = dict(S=[257, 383, 384, 385, 511, 512, 513, 130, 1000, 640], k=[0, 1, 2, 3, 4, 5, 0, 70, 9, 33])


@pytest.mark.parametrize("hq,hkv", [(16, 2), (16, 16)])
def test_fp32_large_tiles(hq, hkv):
    S, k = LARGE["S"], LARGE["k"]
    c = attn_case(hkv, len(S), hq, hkv, 64, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    for r, j in ((2, 1), (7, 0), (7, 69)):
        for pool in ("kpool", "vpool"):
            c[pool][c["page_table"][r, j]] = 0
    want = oracle.attention(**c, n_threads=8)
    for n, (r, j) in enumerate(((2, 1), (7, 0), (7, 69))):
        c["page_table"][r, j] = -1 if n % 2 else sum(k) + 3 + n
    got = run_attn(c)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= F32_TOL


def test_fp32_pages_of_more_than_64_tiles():
    # a wavefront of the large tiles holds the page ids of 64 key tiles (4096 keys) at a time
    S, k = [260, 1030, 2900], [300, 0, 513]
    c = attn_case(3, 3, 16, 1, 64, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    rows = (np.repeat([0, 1, 2], 40).astype(np.int32), np.tile(np.arange(40) % 16, 3).astype(np.int32),
            np.concatenate([np.linspace(0, s - 1, 40) for s in S]).astype(np.int32))
    want = oracle.attention(**c, rows=rows, n_threads=8)
    got = run_attn(c)
    at = np.array([c["q_off"][r] + i for r, i in zip(rows[0], rows[2])])
    assert np.abs(got[at, rows[1]] - want.reshape(len(at), -1)).max() <= F32_TOL


@pytest.mark.parametrize("large,d", [(False, 64), (False, 128), (True, 64)])
def test_fp32_values_without_pieces(large, d):
    # what is not finite, or too large for bf16, reaches the rows that see it and no others
    S, k = (LARGE["S"], LARGE["k"]) if large else ([70, 5, 40], [3, 1, 0])
    n = len(S)
    c = attn_case(31, n, 16, 2, d, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    c["q"] = c["q"].abs() + 0.1
    r = 0 if not large else 8
    first = int(c["q_off"][r])
    nan_row, inf_row, big_row = S[r] - 3, S[r] - 20, S[r] - 30
    low = int(c["page_table"][r, 1 if not large else 4]) if k[r] > 1 else None
    if low is not None:
        c["kpool"][low] = float("-inf")               # no weight
    c["vnew"][first + big_row, :, 3] = 3.4e38         # finite, rounds to infinity as bf16
    want = oracle.attention(**c, n_threads=8)
    c["vnew"][first + nan_row, 0] = float("nan")
    c["vnew"][first + inf_row, 1, 5] = float("inf")
    got = run_attn(c)
    scale = np.maximum(1.0, np.abs(want))             # the large value: relative, as its weight is
    err = np.abs(got - want) / scale
    G = 8
    rows, heads = np.arange(first, first + S[r]), np.arange(16)
    clean = np.ones(got.shape, bool)
    clean[first + nan_row: first + S[r], :G] = False
    clean[first + inf_row: first + S[r], G:, 5] = False
    assert np.isfinite(got[clean]).all() and err[clean].max() <= F32_TOL
    assert np.isnan(got[first + nan_row: first + S[r], :G]).all()
    assert np.isposinf(got[first + inf_row: first + S[r], G:, 5]).all()


# bf16, items split along their keys (few work items behind many keys): 1, 2, 3 .. key tiles a part, parts that end before
# and behind the reused prefix, short first row tiles, rows of several requests.  Tolerance of the unsplit kernel.
SPLIT = [
    (8, 2, [1], [100]), (8, 2, [137], [187]), (16, 8, [64, 5], [64, 300]), (64, 8, [263], [120]), (4, 4, [300], [90]),
    (4, 2, [200, 1, 0, 129], [33, 250, 4, 100]), (3, 1, [70], [160]), (8, 1, [1500], [0]), (32, 8, [700], [10]),
    (32, 8, [40] * 20, [40] * 20),
]


@pytest.mark.parametrize("case", range(len(SPLIT)))
def test_bf16_split_along_the_keys(case):
    hq, hkv, S, k = SPLIT[case]
    c = attn_case(60 + case, len(S), hq, hkv, 128, torch.bfloat16, max(k) + 1, S, k, n_pages=sum(k) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 2e-2
    if max(k) > 40:   # pages outside the pool read as zeros in every part
        r = int(np.argmax(k))
        for j in (0, k[r] // 2, k[r] - 1):
            c["kpool"][c["page_table"][r, j]] = 0
            c["vpool"][c["page_table"][r, j]] = 0
        want = oracle.attention(**c, n_threads=8)
        c["page_table"][r, [0, k[r] // 2, k[r] - 1]] = [-1, sum(k) + 3, -5]
        assert np.abs(run_attn(c) - want).max() <= 2e-2


def test_bf16_split_parts_with_their_own_references():
    # scores that differ by hundreds of exp2 units between the parts: the merge keeps only the largest
    c = attn_case(77, 1, 8, 2, 128, torch.bfloat16, 130, [100], [128], n_pages=131)
    for j in range(128):
        c["kpool"][c["page_table"][0, j]] *= (j % 40) * 2.0
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.abs(got - want).max() <= 2e-2 * max(1.0, np.abs(want).max())   # output rounding at values above 1


@pytest.mark.parametrize("hq,hkv", [(8, 1), (4, 1), (16, 2)])
def test_bf16_work_list_of_many_requests(hq, hkv):
    # more requests than the list is made of at a time, lengths in no order, some alike, some empty; tiles of 32 and 64 rows
    g = np.random.default_rng(hq)
    S = g.choice([0, 1, 2, 5, 17, 31, 32, 33, 64, 65], 1500, p=[.3, .3, .1, .1, .05, .03, .03, .03, .03, .03])
    S[[3, 700, 1400]] = 150, 97, 130
    k = g.integers(0, 3, 1500)
    k[[3, 700, 1023, 1024]] = 20, 9, 30, 2
    c = attn_case(91, 1500, hq, hkv, 128, torch.bfloat16, 31, S, k, n_pages=int(k.sum()) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 2e-2


# Eight query heads per kv head: tiles of 32 rows of eight heads or of 64 rows of four, whichever the lengths favour.  One request
# or several that fill less than the chip; tables wider than what is reused; enough
# to fill the chip with short and with ragged requests, with the last tile on either side of 32 rows.
EIGHT = [
    (64, 8, [1], [2], 600), (16, 2, [40, 64, 65, 33], [0, 1, 2, 9], 700), (8, 1, [64, 200], [7, 3], 10), (16, 1, [1] * 300, [1] * 300, 1),
    (64, 8, [20] * 40, [3] * 40, 3), (16, 2, [97, 31, 160, 0, 1] * 40, [1, 0, 2, 3, 1] * 40, 3), (64, 8, [300] * 3, [20] * 3, 20),
    (32, 2, [33] * 200, [2] * 200, 2),
]


@pytest.mark.parametrize("case", range(len(EIGHT)))
@pytest.mark.parametrize("static", [False, True])
def test_bf16_eight_heads(case, static):
    from paper_2508_08438_amd import binding as skv
    hq, hkv, S, k, width = EIGHT[case]
    c = attn_case(80 + case, len(S), hq, hkv, 128, torch.bfloat16, width, S, k, n_pages=sum(k) + 3)
    if static:
        x = {n: (v if torch.is_tensor(v) else torch.from_numpy(v)).to("cuda:0") for n, v in c.items()}
        out = torch.full_like(x["q"], 7.0)
        skv.skv_prefill_attn_static(skv.attn_desc(hq, hkv, 128, "bf16"), x["q"], x["knew"], x["vnew"], x["q_off"], x["kpool"],
                                    x["vpool"], x["matched_len"], x["page_table"], width, out)
        got = out.double().cpu().numpy()
    else:
        got = run_attn(c)
    want = oracle.attention(**c, n_threads=16)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 2e-2


def _run_with(c, workspace_bytes):
    from paper_2508_08438_amd import binding as skv
    dev = "cuda:0"
    x = {n: (v if torch.is_tensor(v) else torch.from_numpy(v)).to(dev) for n, v in c.items()}
    desc = skv.attn_desc(x["q"].shape[1], x["kpool"].shape[2], 128, torch.bfloat16)
    full = skv.skv_prefill_attn_workspace_size(desc, len(c["matched_len"]), x["q"].shape[0])
    ws = torch.zeros(full if workspace_bytes is None else workspace_bytes, dtype=torch.uint8, device=dev)
    out = torch.full_like(x["q"], 7.0)
    skv.skv_prefill_attn(desc, x["q"], x["knew"], x["vnew"], x["q_off"], x["kpool"], x["vpool"], x["matched_len"],
                         x["page_table"], x["page_table"].shape[1], out, ws)
    torch.cuda.synchronize()
    return out.double().cpu().numpy(), full


@pytest.mark.parametrize("hq,hkv", [(8, 2), (8, 1)])
def test_bf16_plain_work_list_is_enough(hq, hkv):
    from paper_2508_08438_amd import binding as skv
    c = attn_case(13, 2, hq, hkv, 128, torch.bfloat16, 150, [70, 9], [150, 40], n_pages=200)
    want = oracle.attention(**c, n_threads=8)
    # item count, page of zeros, a record of 32 bytes for each of 79 / 64 (rows per tile of four heads) + 2 per request
    plain = 256 + 16 * hkv * 256 + 256
    got, full = _run_with(c, plain)
    assert full > plain and np.abs(got - want).max() <= 2e-2
    with pytest.raises(skv.SkvError) as e:
        _run_with(c, plain - 1)
    assert e.value.code == skv.SKV_ENOMEM


@pytest.mark.parametrize("hq,hkv", [(32, 8), (64, 8), (8, 1)])
def test_bf16_workspace_of_a_larger_batch(hq, hkv):
    # a server's one buffer, sized for its largest batch: small batches are split along their keys as with a buffer of their own
    from paper_2508_08438_amd import binding as skv
    largest = skv.skv_prefill_attn_workspace_size(skv.attn_desc(hq, hkv, 128, "bf16"), 256, 65536)
    for S, k in (([137], [187]), ([64, 9, 300], [150, 40, 7])):
        c = attn_case(13, len(S), hq, hkv, 128, torch.bfloat16, max(k), S, k, n_pages=sum(k) + 1)
        own, _ = _run_with(c, None)
        got, _ = _run_with(c, largest)
        plain, _ = _run_with(c, 256 + 16 * hkv * 256 + 1024)
        assert np.array_equal(got, own)
        assert not np.array_equal(got, plain)     # (parts round their own way: so there were parts)


@pytest.mark.parametrize("split", [True, False])
def test_bf16_runs_of_keys_without_weight(split):
    # scores of -infinity over the first pages, over whole parts, and over the new keys of one request
    c = attn_case(14, 2, 8, 2, 128, torch.bfloat16, 130, [70, 40], [128, 100], n_pages=230)
    c["q"] = c["q"].abs() + 0.01
    for r, pages in ((0, range(0, 4)), (0, range(20, 90)), (1, range(96, 100))):
        for j in pages:
            c["kpool"][c["page_table"][r, j]] = float("-inf")
    c["knew"][70:] = float("-inf")
    got, _ = _run_with(c, None if split else 256 + 16 * 2 * 256 + 256)
    want = oracle.attention(**c, n_threads=8)
    assert np.isfinite(want).all() and np.abs(got - want).max() <= 2e-2
