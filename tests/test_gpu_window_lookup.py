"""The lookup that opens a monitoring window and leaves its counters to the step's second call, against a reset and a lookup."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2508_08438_amd import binding as skv
from paper_2508_08438_amd import inputs, pipeline

pytestmark = pytest.mark.gpu


def _session(seed=3, **k):
    w = inputs.small_random(seed=seed, **{**dict(n_seq=8, max_blocks=24, n_req=12, vocab=50, n_tenants=100,
                                                 attn=inputs.AttnShape(8, 2, 128, "bf16")), **k})
    s = pipeline.Session(w)
    s.prepare()
    return s


def _dirty(s):
    """Counters of an earlier lookup stand in every block that it matched."""
    for _ in range(3):
        skv.skv_match(s.tree, s.req_off, s.req_tokens, s.req_tenant, s.max_blocks, s.matched_len, s.page_table)


def _want(s):
    s.match()
    want = s.counters()
    assert want[0].sum() > 0
    return want, [x.cpu().clone() for x in (s.matched_len, s.page_table)]


def _window(s):
    return skv.skv_match_window(s.tree, s.req_off, s.req_tokens, s.req_tenant, s.max_blocks, s.matched_len, s.page_table, s.records)


# arguments that are refused: of the offsets, of the gather, of the attention, before anything is launched
@pytest.mark.parametrize("bad", [dict(q_off=None), dict(req_off=None), dict(ctx_off=None), dict(cap=-1), dict(desc=None), dict(q=None), dict(ws_bytes=0)])
def test_refused_step_has_counted(bad):
    s = _session()
    want, _ = _want(s)
    _dirty(s)
    assert _window(s)
    p = lambda t: t.data_ptr()
    a = dict(desc=C.byref(s.desc), n_req=s.w.n_req, req_off=p(s.req_off), q=p(s.q), knew=p(s.knew), vnew=p(s.vnew), q_off=p(s.q_off),
             rows=s.q.shape[0], kpool=p(s.kpool), vpool=p(s.vpool), n_pages=s.kpool.shape[0], matched=p(s.matched_len),
             table=p(s.page_table), mb=s.max_blocks, out=p(s.out), ctx_off=p(s.ctx_off), kctx=p(s.kctx), vctx=p(s.vctx),
             cap=s.kctx.shape[0], tree=s.tree.handle, tenant=p(s.req_tenant), records=p(s.records), ws=p(s.workspace),
             ws_bytes=s.workspace.numel(), stream=torch.cuda.current_stream().cuda_stream)
    assert skv.lib().skv_prefill_step(*{**a, **bad}.values()) in (skv.SKV_EINVAL, skv.SKV_ENOMEM)
    assert all(np.array_equal(x, y) for x, y in zip(want, s.counters()))


# workgroups behind the requests' clear the counters, 256 records each and 4096 of them at most: trees on both sides of one workgroup, of
# several, and of the most there are (four records and more each)
@pytest.mark.parametrize("n_seq,max_blocks", [(1, 1), (8, 24), (13, 40), (64, 60), (300, 40)])
def test_window_is_reset_and_lookup(n_seq, max_blocks):
    s = _session(seed=n_seq, n_seq=n_seq, max_blocks=max_blocks, p_sens=0.0)
    want, state = _want(s)
    _dirty(s)
    s.matched_len.fill_(-7)
    s.page_table.fill_(-7)
    assert _window(s)
    assert all(torch.equal(a, b.cpu()) for a, b in zip(state, (s.matched_len, s.page_table)))
    assert not any(c.any() for c in s.counters())                 # cleared, not yet counted
    skv.skv_prefill_step(s.desc, s.req_off, s.q, s.knew, s.vnew, s.q_off, s.kpool, s.vpool, s.matched_len, s.page_table, s.max_blocks, s.out,
                         s.ctx_off, s.kctx, s.vctx, s.workspace, tree=s.tree, req_tenant=s.req_tenant, records=s.records)
    assert all(np.array_equal(a, b) for a, b in zip(want, s.counters()))


def test_largest_grid_clears_every_record():
    """More blocks than 4096 workgroups have threads: one request that matches a run of them, and all others' counters."""
    n = 4096 * 256 + 300
    g = np.random.default_rng(1)
    tokens = g.integers(0, 30000, n * 16, dtype=np.int32)
    tree = skv.skv_tree_build(tokens, np.array([0, n * 16], np.int64), np.zeros(n, np.uint8), np.zeros(n, np.int32),
                              np.arange(n, dtype=np.int32), 4, n, device="cuda:0")
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    m = 2000
    i32 = lambda *k: torch.zeros(k, dtype=torch.int32, device="cuda:0")
    hit, users = i32(n), i32(n)
    whole = (dev(np.array([0, n * 16], np.int32)), dev(tokens), i32(1))
    matched, table = i32(1), i32(1, n)
    skv.skv_match(tree, *whole, n, matched, table)
    skv.skv_counters_read(tree, hit, users)
    assert int(matched) == n * 16 and int(hit.min()) == 1 == int(users.min())
    part = (dev(np.array([0, m * 16], np.int32)), dev(tokens[: m * 16]), i32(1))
    assert skv.skv_match_window(tree, *part, m, matched, i32(1, m), i32(1, m))
    skv.skv_counters_read(tree, hit, users)
    assert int(matched) == m * 16 and not hit.any() and not users.any()


# what is left to the two calls: a tree with per-tenant copies, no room for records, more than 512 requests, none
@pytest.mark.parametrize("case", ["copies", "no records", "513 requests", "no requests"])
def test_window_falls_back(case):
    s = _session(n_req=513 if case == "513 requests" else 12)
    if case == "copies":
        w = s.w
        left = (np.diff(w.req_off) - s.matched_len.cpu().numpy()) // 16
        pages = np.where(np.arange(max(int(left.max()), 1))[None, :] < left[:, None], 0, -1).astype(np.int32)
        n_new = int((pages == 0).sum())
        pages[pages == 0] = w.n_pages + np.arange(n_new)
        s.tree = skv.skv_tree_build(w.seq_tokens, w.seq_off, w.blk_sensitive, w.blk_owner, w.blk_page, w.n_tenants, w.n_pages + n_new,
                                    reserve_blocks=n_new + 64)
        end = torch.zeros_like(s.matched_len)
        skv.skv_match(s.tree, s.req_off, s.req_tokens, s.req_tenant, s.max_blocks, s.matched_len, s.page_table, path_end=end)
        skv.skv_tree_insert(s.tree, w.req_off, w.req_tokens, w.req_tenant, s.matched_len.cpu().numpy(), pages, private_copies=True,
                            path_end=end.cpu().numpy())
    n = s.tree.info()["n_in_blocks"]

    def counters():
        hit, users = (torch.zeros(n, dtype=torch.int32, device="cuda:0") for _ in "hu")
        skv.skv_counters_read(s.tree, hit, users)
        return hit.cpu(), users.cpu()
    s.match()
    want, state = counters(), [x.cpu().clone() for x in (s.matched_len, s.page_table)]
    _dirty(s)
    left = C.c_int32(7)
    p = lambda t: t.data_ptr()
    n_req = 0 if case == "no requests" else s.w.n_req
    assert skv.lib().skv_match_window(s.tree.handle, n_req, p(s.req_off), p(s.req_tokens), p(s.req_tenant), s.max_blocks, p(s.matched_len),
                                      p(s.page_table), None if case == "no records" else p(s.records), C.byref(left),
                                      torch.cuda.current_stream().cuda_stream) == skv.SKV_OK
    assert left.value == 0
    got = counters()
    if case == "no requests":
        assert not got[0].any() and not got[1].any()
        return
    assert want[0].any() and all(torch.equal(a, b) for a, b in zip(want, got))
    assert all(torch.equal(a, b.cpu()) for a, b in zip(state, (s.matched_len, s.page_table)))
