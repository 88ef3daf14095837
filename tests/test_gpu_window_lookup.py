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
