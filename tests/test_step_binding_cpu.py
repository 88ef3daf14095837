"""The binding of the step's second call refuses tensors of the wrong type or size before it takes their addresses; host tensors, which
it refuses last, stand in for device memory."""
import pytest
import torch

from paper_2508_08438_amd import binding as skv
from test_step_call_cpu import _lib

i32, i64, f = torch.int32, torch.int64, torch.bfloat16
z = torch.zeros


def _args():
    return dict(desc=skv.attn_desc(8, 2, 128, "bf16"), req_off=z(3, dtype=i32), q=z(5, 8, 128, dtype=f), knew=z(5, 2, 128, dtype=f),
                vnew=z(5, 2, 128, dtype=f), q_off=z(3, dtype=i32), kpool=z(4, 16, 2, 128, dtype=f), vpool=z(4, 16, 2, 128, dtype=f),
                matched_len=z(2, dtype=i32), page_table=z(2, 3, dtype=i32), max_blocks=3, out=z(5, 8, 128, dtype=f),
                ctx_off=z(3, dtype=i64), kctx=z(32, 2, 128, dtype=f), vctx=z(32, 2, 128, dtype=f), workspace=z(64, dtype=torch.uint8),
                tree=object(), req_tenant=z(2, dtype=i32), records=z(2, 3, dtype=i32))


@pytest.mark.parametrize("bad", [dict(q_off=z(3, dtype=i64)), dict(req_off=z(3, dtype=i64)), dict(matched_len=z(2, dtype=i64)),
                                 dict(page_table=z(2, 3, dtype=i64)), dict(page_table=z(5, dtype=i32)), dict(records=z(2, 3, dtype=i64)),
                                 dict(records=z(5, dtype=i32)), dict(req_tenant=z(2, dtype=i64)), dict(req_tenant=z(1, dtype=i32)),
                                 dict(tree=None), dict(q_off=z(2, dtype=i32)), dict(ctx_off=z(3, dtype=i32))])
def test_step_binding_refuses(bad):
    _lib()
    with pytest.raises(AssertionError) as e:
        skv.skv_prefill_step(**{**_args(), **bad})
    assert "device tensor" not in str(e.value)


def test_step_binding_takes_the_rest():
    _lib()
    for a in (_args(), {**_args(), "tree": None, "req_tenant": None, "records": None}):
        with pytest.raises(AssertionError, match="device tensor"):
            skv.skv_prefill_step(**a)
