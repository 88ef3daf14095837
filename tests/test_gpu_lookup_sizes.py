"""Sizes at which the kernels around the lookup change chunk: suffix offsets of more requests than one chunk, counters and
read-backs of a slab with room to spare, before and after evictions and compaction."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08438_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _skv():
    from paper_2508_08438_amd import binding
    return binding


@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 256, 257, 4095, 4096, 4097, 9001])
def test_suffix_offsets(n):
    skv = _skv()
    g = np.random.default_rng(n)
    length = g.integers(0, 50, n)
    off = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    matched = g.integers(0, 60, n).astype(np.int32)          # more than the length now and then: counts as none left
    out = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV)
    skv.skv_suffix_offsets(torch.from_numpy(off).to(DEV), torch.from_numpy(matched).to(DEV), out)
    want = np.concatenate([[0], np.cumsum(np.maximum(length - matched, 0))])
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("reserve", [0, 1, 777])
def test_counters_of_a_slab_with_room(reserve):
    skv = _skv()
    w = inputs.small_random(seed=21 + reserve, n_seq=12, max_blocks=40, n_req=90, vocab=40, n_tenants=128)
    tree = skv.skv_tree_build(w.seq_tokens, w.seq_off, w.blk_sensitive, w.blk_owner, w.blk_page, w.n_tenants, w.n_pages,
                              device=DEV, reserve_blocks=reserve)
    ref = oracle.OracleTree.from_workload(w)
    dev = lambda x: torch.from_numpy(x).to(DEV)
    i32 = lambda n: torch.full((max(n, 1),), -7, dtype=torch.int32, device=DEV)
    mb = max(w.max_blocks, 1)
    ml, pt = i32(w.n_req), i32(w.n_req * mb).view(w.n_req, mb)
    for _ in range(2):
        skv.skv_match(tree, dev(w.req_off), dev(w.req_tokens), dev(w.req_tenant), mb, ml, pt)
        ref.match(w.req_off, w.req_tokens, w.req_tenant, mb)
    want_hit, want_users = (x.copy() for x in ref.counters())
    n = w.n_in_blocks

    def read():
        hit, users = i32(n), i32(n)
        skv.skv_counters_read(tree, hit, users)
        priv = torch.full((max(n, 1),), 7, dtype=torch.uint8, device=DEV)
        pre, upre = i32(n), i32(n)
        skv.skv_block_state_read(tree, priv, pre, upre)
        return [x.cpu().numpy()[:n] for x in (hit, users, priv, pre, upre)]

    hit, users, priv, pre, upre = read()
    assert np.array_equal(hit.view(np.uint32), want_hit) and np.array_equal(users.view(np.uint32), want_users)
    assert not pre.any() and not upre.any()
    created = priv != 255                                     # the rest found their block cached already: no entry of their own
    assert not hit[~created].any() and np.array_equal(priv[created], w.blk_sensitive[created])
    skv.skv_window_roll(tree, skv.rdr_policy(tau=(1, 100), min_hits=1 << 30))
    h2, u2, p2, pre, upre = read()
    assert not h2.any() and not u2.any() and np.array_equal(p2, priv)
    assert np.array_equal(pre, hit) and np.array_equal(upre, users)
    # evicted entries read as none; the others keep their values through a compaction
    ids, _ = skv.skv_evict(tree, int(created.sum()) // 3)
    keep = created.copy()
    keep[ids] = False
    _, _, p3, pre3, upre3 = read()
    assert (p3[~keep] == 255).all() and not pre3[~keep].any() and np.array_equal(pre3[keep], pre[keep])
    id_map = skv.skv_tree_compact(tree)
    assert (id_map[keep] >= 0).all() and (id_map[~keep] < 0).all()
    n = int(keep.sum())
    _, _, p4, pre4, upre4 = read()
    assert np.array_equal(p4, priv[keep]) and np.array_equal(pre4, pre[keep]) and np.array_equal(upre4, upre[keep])
