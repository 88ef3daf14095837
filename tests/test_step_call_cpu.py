"""The step's two calls without a GPU: malformed arguments are refused before any device work."""
import ctypes as C

import pytest

from paper_2508_08438_amd import binding as skv

P = 4096   # stands for a pointer that is never followed
OK = dict(n_req=1, req_off=P, q=P, knew=P, vnew=P, q_off=P, rows=4, kpool=P, vpool=P, n_pages=2, matched=P, table=P, mb=1, out=P, ctx_off=P,
          kctx=P, vctx=P, cap=16, tree=None, tenant=None, records=None, ws=None, ws_bytes=0)


def _lib():
    import os
    if not os.path.exists(skv.LIB_PATH):
        from paper_2508_08438_amd.build import build_lib
        build_lib()
    return skv.lib()


@pytest.mark.parametrize("bad", [dict(n_req=-1), dict(q_off=None), dict(req_off=None), dict(matched=None), dict(records=P), dict(records=P, tree=P),
                                 dict(ctx_off=None), dict(kpool=None), dict(kctx=P + 4), dict(cap=-1), dict(table=None), dict(mb=-1), dict(desc=None)])
def test_step_refuses(bad):
    desc = skv.attn_desc(8, 2, 128, "bf16")
    a = {**OK, "desc": C.byref(desc), **bad}
    assert _lib().skv_prefill_step(a.pop("desc"), *(a[k] for k in OK), None) == skv.SKV_EINVAL


@pytest.mark.parametrize("args", [(None, 1, P, P, P, 1, P, P, P), (P, -1, P, P, P, 1, P, P, P), (P, 1, P, P, P, -1, P, P, P)])
def test_lookup_of_a_step_refuses(args):
    assert _lib().skv_match_window(*args, C.byref(C.c_int32()), None) == skv.SKV_EINVAL
