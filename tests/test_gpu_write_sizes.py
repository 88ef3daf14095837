"""Insertion, eviction and compaction whose transfers do not fit the pinned staging memory (1 MiB), and ones that do, against
the oracle: results of the calls, and what lookups find afterwards."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
B = 16


def test_transfers_larger_than_the_stage():
    from paper_2508_08438_amd import binding as skv
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    g = np.random.default_rng(12)
    P, nb = 3000, 100                                   # 300 k blocks: 1.2 MB of epochs
    n, spare = P * nb, 20000
    toks = g.integers(0, 50000, P * nb * B, dtype=np.int32)
    off = np.arange(P + 1, dtype=np.int64) * nb * B
    args = (toks, off, np.zeros(n, np.uint8), g.integers(0, 4, n).astype(np.int32), g.permutation(n + spare)[:n].astype(np.int32))
    tree = skv.skv_tree_build(*args, 4, n + spare, device="cuda:0", reserve_blocks=spare)
    ref = oracle.OracleTree(*args)
    pages = np.setdiff1d(np.arange(n + spare), args[4]).astype(np.int32)

    def lookup(which, extra=None):
        reqs = [toks[w * nb * B: (w * nb + int(g.integers(1, nb + 1))) * B] for w in which] + (extra or [])
        x, o = np.concatenate(reqs), np.concatenate([[0], np.cumsum([len(r) for r in reqs])]).astype(np.int32)
        ten = g.integers(0, 4, len(reqs)).astype(np.int32)
        mb = max(len(r) for r in reqs) // B
        ml, pt = dev(np.zeros(len(reqs), np.int32)), dev(np.zeros((len(reqs), mb), np.int32))
        skv.skv_match(tree, dev(o), dev(x), dev(ten), mb, ml, pt)
        want_ml, want_pt = ref.match(o, x, ten, mb)
        assert np.array_equal(ml.cpu().numpy(), want_ml) and np.array_equal(pt.cpu().numpy(), want_pt)

    def epoch(e):
        skv.skv_set_epoch(tree, e)
        ref.set_epoch(e)

    epoch(1)
    lookup(g.integers(0, P, 500))
    epoch(2)
    R, add = 200, 70                                    # 14 k new blocks: 1.2 MB of records
    new = [g.integers(0, 50000, add * B, dtype=np.int32) for _ in range(R)]
    o = (np.arange(R + 1) * add * B).astype(np.int32)
    ten, zero = g.integers(0, 4, R).astype(np.int32), np.zeros(R, np.int32)
    table = pages[: R * add].reshape(R, add)
    first, k = skv.skv_tree_insert(tree, o, np.concatenate(new), ten, zero, table, private_copies=True)
    o_first, o_k = ref.insert(o, np.concatenate(new), ten, zero, table, private_copies=True)
    assert np.array_equal(first, o_first) and np.array_equal(k, o_k) and k.sum() == R * add
    lookup(g.integers(0, P, 100), new)
    for n_want in (5000, 150000):                       # a list that fits, one that does not
        ids, pg = skv.skv_evict(tree, n_want)
        o_ids, o_pg = ref.evict(n_want)
        assert np.array_equal(ids, o_ids) and np.array_equal(pg, o_pg)
        epoch(3)
        lookup(g.integers(0, P, 300), new)
    id_map = skv.skv_tree_compact(tree)
    lookup(g.integers(0, P, 300), new)
    ids, pg = skv.skv_evict(tree, 1000)
    o_ids, o_pg = ref.evict(1000)
    assert np.array_equal(ids, id_map[o_ids]) and np.array_equal(pg, o_pg)
    lookup(g.integers(0, P, 300), new)
