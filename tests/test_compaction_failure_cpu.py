"""A compaction whose copies, launches or waits fail, without a GPU (see test_write_side_cpu)."""
import ctypes as C

import numpy as np

from paper_2508_08438_amd import inputs
from test_oracle_insert import make_round
from test_write_side_cpu import B, HostTree, _p, lib  # noqa: F401


def _info(lib, t):
    x = [C.c_int64() for _ in range(3)]
    lib.skv_tree_info(t.h, *map(C.byref, x))
    return [v.value for v in x]


def test_a_compaction_that_fails_changes_nothing(lib):  # noqa: F811
    """Every copy, launch and wait of a compaction fails once: the tree's state on the host is what it was, so with the slab put back the
    tree goes on like one that never tried."""
    lib.host_refuse_pinned(1)
    try:
        w = inputs.small_random(seed=5, n_seq=12, max_blocks=30, vocab=30, n_tenants=3)
        pages = w.n_pages + 400
        trees = [HostTree(lib, w, pages, 500) for _ in "ab"]      # the second one never fails
        bytes_of = lambda t: t.slab[(-t.slab.ctypes.data) % 256:][: len(t.slab) - 256]
        info = lambda t: _info(lib, t)
        g = np.random.default_rng(5)
        earlier = [w.req_tokens[w.req_off[r]: w.req_off[r + 1]] for r in range(w.n_req)]
        free, failed = list(range(w.n_pages, pages)), []
        for rnd in range(3):
            for t in trees:
                lib.skv_set_epoch(t.h, rnd + 1)
            reqs, off, toks, tenants = make_round(g, earlier, 30, 3, 10, None)
            toks = toks if len(toks) else np.zeros(1, np.int32)
            mb = max(max(len(x) // B for x in reqs), 1)
            new = np.full((10, mb), -1, np.int32)
            for r, x in enumerate(reqs):
                for j in range(len(x) // B):
                    new[r, j] = free.pop()
            got = [t.insert(off, toks, tenants, np.zeros(10, np.int32), new) for t in trees]
            assert got[0][0] == got[1][0] == 0 and all(np.array_equal(a, b) for a, b in zip(got[0][1:], got[1][1:]))
            n, prot = info(trees[0])[1] // 4, g.choice(40, 5)
            got = [t.evict(n, prot) for t in trees]
            assert got[0][0] == got[1][0] == 0 and all(np.array_equal(a, b) for a, b in zip(got[0][1:], got[1][1:]))
            before, was = info(trees[0]), bytes_of(trees[0]).copy()
            for k in range(1, 200):
                id_map, after = np.full(before[2], -7, np.int32), C.c_int64(-7)
                lib.host_fail_in(C.c_long(k))
                rc = lib.skv_tree_compact(trees[0].h, _p(id_map), C.byref(after), None)
                lib.host_fail_in(C.c_long(0))
                if rc == 0:
                    break
                assert (id_map == -7).all() and after.value == -7 and info(trees[0]) == before, k
                bytes_of(trees[0])[:] = was
            rc, want = trees[1].compact()
            assert rc == 0 and np.array_equal(id_map, want) and info(trees[0]) == info(trees[1])
            assert np.array_equal(bytes_of(trees[0]), bytes_of(trees[1]))
            failed.append(k - 1)
            earlier += reqs
        assert max(failed) == 29, failed   # ten spans down, a wait, sixteen up, the fills and a wait
        left = [t.evict(info(t)[1] + 5, []) for t in trees]
        assert left[0][0] == left[1][0] == 0 and all(np.array_equal(a, b) for a, b in zip(left[0][1:], left[1][1:]))
        for t in trees:
            t.destroy()
    finally:
        lib.host_fail_in(C.c_long(0))
        lib.host_refuse_pinned(0)
