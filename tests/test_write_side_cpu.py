"""The host side of insertion, eviction and compaction against the oracle, without a GPU: skv_tree.hip linked with
host_runtime.cpp.  Without pinned memory every transfer is a copy the stand-in carries out, so the whole state is real."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import OracleTree
from paper_2508_08438_amd import build, inputs
from paper_2508_08438_amd.binding import TreeDesc
from test_oracle_insert import make_round

B = 16
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    obj, out = str(d / "tree.o"), str(d / "libtree_host.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    for cmd in ([hipcc, *[f for f in build.FLAGS if f != "-shared"], "-c", "-I", build.INCLUDE, "-I", build.CSRC, "-o", obj,
                 os.path.join(build.CSRC, "skv_tree.hip")],
                ["g++", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", out, obj, os.path.join(HERE, "host_runtime.cpp")]):
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout
    l = C.CDLL(out)
    for f in ("host_calls", "host_pinned"):
        getattr(l, f).restype = C.c_long
    return l


def _p(a):
    return C.c_void_p(a.ctypes.data)


class HostTree:
    def __init__(self, lib, w, n_pages, reserve):
        self.lib = lib
        a = [np.ascontiguousarray(w.seq_off, np.int64), np.ascontiguousarray(w.seq_tokens, np.int32),
             np.ascontiguousarray(w.blk_sensitive, np.uint8), np.ascontiguousarray(w.blk_owner, np.int32),
             np.ascontiguousarray(w.blk_page, np.int32)]
        d = TreeDesc(B, w.n_tenants, n_pages, len(a[0]) - 1, *(_p(x) for x in a))
        size = C.c_size_t()
        assert lib.skv_tree_size_for_capacity(C.c_int64(len(a[4]) + reserve), C.byref(size)) == 0
        self.slab = np.zeros(size.value + 256, np.uint8)
        self.h = C.c_void_p()
        base = (self.slab.ctypes.data + 255) // 256 * 256
        assert lib.skv_tree_build(C.byref(d), C.c_void_p(base), size, None, C.byref(self.h)) == 0

    def insert(self, off, toks, tenants, mlen, pages):
        first, n = np.zeros(len(tenants), np.int32), np.zeros(len(tenants), np.int32)
        rc = self.lib.skv_tree_insert(self.h, len(tenants), _p(off), _p(toks), _p(tenants), _p(mlen), _p(pages), pages.shape[1],
                                      1, None, _p(first), _p(n), None)
        return rc, first, n

    def evict(self, n, protect):
        ids, pages, k = np.zeros(max(n, 1), np.int32), np.zeros(max(n, 1), np.int32), C.c_int64()
        protect = np.ascontiguousarray(protect, np.int32)
        rc = self.lib.skv_evict(self.h, C.c_int64(n), _p(protect), C.c_int64(len(protect)), _p(ids), _p(pages), C.byref(k), None)
        return rc, ids[: k.value], pages[: k.value]

    def compact(self):
        n_in = C.c_int64()
        self.lib.skv_tree_info(self.h, None, None, C.byref(n_in))
        id_map, after = np.full(max(n_in.value, 1), -1, np.int32), C.c_int64()
        return self.lib.skv_tree_compact(self.h, _p(id_map), C.byref(after), None), id_map[: n_in.value]

    def destroy(self):
        self.lib.skv_tree_destroy(self.h)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_write_calls_need_no_pinned_memory(lib, seed):
    lib.host_refuse_pinned(1)
    try:
        w = inputs.small_random(seed=seed, n_seq=10, max_blocks=30, vocab=30, n_tenants=3)
        pages = w.n_pages + 600
        tree, ref = HostTree(lib, w, pages, 700), OracleTree.from_workload(w)
        g = np.random.default_rng(seed)
        earlier = [w.req_tokens[w.req_off[r]: w.req_off[r + 1]] for r in range(w.n_req)]
        free = list(range(w.n_pages, pages))
        new_of = np.arange(10000)                      # the oracle's ids -> this tree's (compaction renumbers)
        for rnd in range(6):
            lib.skv_set_epoch(tree.h, rnd + 1)
            ref.set_epoch(rnd + 1)
            reqs, off, toks, tenants = make_round(g, earlier, 30, 3, 10, None)
            toks = toks if len(toks) else np.zeros(1, np.int32)
            mb = max(max(len(x) // B for x in reqs), 1)
            mlen, _ = ref.match(off, toks, tenants, mb, update=False)
            new = np.full((10, mb), -1, np.int32)
            for r, x in enumerate(reqs):
                for j in range(len(x) // B - mlen[r] // B):
                    new[r, j] = free.pop()
            n_before = ref.n_in_blocks
            rc, first, n = tree.insert(off, toks, tenants, mlen, new)
            o_first, o_n = ref.insert(off, toks, tenants, mlen, new, private_copies=True)
            assert rc == 0 and np.array_equal(first, o_first) and np.array_equal(n, o_n)
            n_in = C.c_int64()
            lib.skv_tree_info(tree.h, None, None, C.byref(n_in))
            new_of[n_before: ref.n_in_blocks] = n_in.value - (ref.n_in_blocks - n_before) + np.arange(ref.n_in_blocks - n_before)
            prot = g.choice(ref.n_in_blocks, 5)
            rc, ids, pg = tree.evict(ref.n_blocks // 4, new_of[prot][new_of[prot] >= 0])
            o_ids, o_pg = ref.evict(ref.n_blocks // 4, prot)
            assert rc == 0 and np.array_equal(ids, new_of[o_ids]) and np.array_equal(pg, o_pg)
            if rnd % 2:
                rc, id_map = tree.compact()
                assert rc == 0
                live = np.flatnonzero(new_of[: ref.n_in_blocks] >= 0)
                new_of[live] = id_map[new_of[live]]
            earlier += reqs
        left = ref.n_blocks
        rc, ids, pg = tree.evict(left + 5, [])
        o_ids, o_pg = ref.evict(left + 5)
        assert rc == 0 and len(ids) == left and np.array_equal(ids, new_of[o_ids]) and np.array_equal(pg, o_pg)
        tree.destroy()
    finally:
        lib.host_refuse_pinned(0)


def test_destroying_a_tree_makes_no_runtime_call(lib):
    w = inputs.small_random(seed=4, n_seq=6, max_blocks=10, vocab=30)
    trees = [HostTree(lib, w, w.n_pages, 10) for _ in range(9)]
    for t in trees:
        assert t.evict(1, [])[0] == 0                  # now every tree has pinned memory of its own
    held = lib.host_pinned()
    assert held == 9
    before = lib.host_calls()
    for t in trees:
        t.destroy()
    assert lib.host_calls() == before and lib.host_pinned() == held
    t = HostTree(lib, w, w.n_pages, 10)                # the next one to write takes a piece over and gives most of the rest back
    assert t.evict(1, [])[0] == 0
    assert lib.host_pinned() <= 5
    t.destroy()
