"""Insertions that a full slab refuses, without a GPU (see test_write_side_cpu): nothing of them is left, whichever request found no room."""
import ctypes as C

import numpy as np
import pytest

from paper_2508_08438_amd import inputs
from test_oracle_insert import make_round
from test_write_side_cpu import B, HostTree, _p, lib  # noqa: F401

ENOMEM = -2


def _insert(t, copies, off, toks, tenants, pages):
    n = len(tenants)
    out = np.full((2, n), -9, np.int32)
    mlen = np.zeros(n, np.int32)
    rc = t.lib.skv_tree_insert(t.h, n, _p(off), _p(toks), _p(tenants), _p(mlen), _p(pages), pages.shape[1], copies, None, _p(out[0]),
                               _p(out[1]), None)
    return rc, out


def _slab(t):
    return t.slab[(-t.slab.ctypes.data) % 256:][: len(t.slab) - 256]


def _round(g, earlier, free):
    reqs, off, toks, tenants = make_round(g, earlier, 6, 3, 8, None if g.random() < 0.5 else 3)
    pages = np.full((8, max(max(len(x) // B for x in reqs), 1)), -1, np.int32)
    for r, x in enumerate(reqs):
        n = len(x) // B
        pages[r, :n] = free[sum(len(y) // B for y in reqs[:r]):][:n]
    return reqs, (off, toks if len(toks) else np.zeros(1, np.int32), tenants, pages)


@pytest.mark.parametrize("copies", [0, 1])
@pytest.mark.parametrize("reserve", [0, 1, 5, 17, 30])
def test_a_refused_insertion_leaves_nothing(lib, copies, reserve):  # noqa: F811
    lib.host_refuse_pinned(1)
    try:
        refused = set()
        for seed in range(12):
            g = np.random.default_rng([seed, reserve, copies])
            w = inputs.small_random(seed=seed, n_seq=6, max_blocks=8, vocab=6, n_tenants=3, block_vocab=3 if seed % 2 else None)
            n_pages = w.n_pages + 300
            trees = [HostTree(lib, w, n_pages, reserve) for _ in "ab"]      # the second one is never asked for what does not fit
            free = list(range(w.n_pages, n_pages))
            earlier = [w.req_tokens[w.req_off[r]: w.req_off[r + 1]] for r in range(w.n_req)]
            for rnd in range(8):
                for t in trees:
                    lib.skv_set_epoch(t.h, rnd + 1)
                reqs, a = _round(g, earlier, free)
                was = _slab(trees[0]).copy()
                rc, out = _insert(trees[0], copies, *a)
                if rc == ENOMEM:
                    refused.add(int((out[0] >= 0).sum()))                   # requests that had gone in
                    assert np.array_equal(_slab(trees[0]), was)
                else:
                    rc2, out2 = _insert(trees[1], copies, *a)
                    assert rc == rc2 == 0 and np.array_equal(out, out2)
                    earlier += reqs
                    used = {int(p) for r in range(8) for p in a[3][r, out[0, r]: out[0, r] + out[1, r]]}
                    free = [p for p in free if p not in used]
                got = [trees[0].evict(int(g.integers(0, 12)), [])]
                got.append(trees[1].evict(len(got[0][1]), []))
                assert all(np.array_equal(x, y) for x, y in zip(*got))
                free += [int(p) for p in got[0][2]]
                if rnd % 3 == 2:
                    (rc, m0), (rc2, m1) = (t.compact() for t in trees)
                    assert rc == rc2 == 0 and np.array_equal(m0, m1)
                assert np.array_equal(_slab(trees[0]), _slab(trees[1]))
            for t in trees:
                t.destroy()
        assert len(refused) >= 3 and max(refused) >= 3                       # at the first requests of a batch and behind them
    finally:
        lib.host_refuse_pinned(0)
