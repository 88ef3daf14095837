"""The gather's form for a stream beside the attention: against the plain form at the sizes where it can go wrong, and the step that
uses it against its stages one after the other, replayed from a graph and with an attention call that is refused."""
import numpy as np
import pytest
import torch

from paper_2508_08438_amd import inputs, pipeline
from paper_2508_08438_amd import binding as skv

pytestmark = pytest.mark.gpu
B = 16


# pages of 4 KB (one step of a workgroup), 12, 20, 32, 80 KB (three steps a turn: remainders), odd ones; around a turn of the
# grid, the scan's chunks and the number of requests that takes the plain form
@pytest.mark.parametrize("n_req,hkv,d,dtype", [(1, 8, 128, "bf16"), (2, 1, 128, "bf16"), (255, 3, 128, "bf16"), (256, 5, 128, "bf16"),
                                               (257, 8, 128, "bf16"), (511, 1, 8, "bf16"), (512, 1, 64, "bf16"), (513, 2, 128, "bf16"),
                                               (64, 20, 128, "bf16"), (0, 8, 128, "bf16"), (40, 3, 40, "f32")])
def test_beside_is_the_plain_gather(n_req, hkv, d, dtype):
    g = np.random.default_rng(n_req + hkv)
    mb = 300 if n_req <= 2 else 9
    blocks = g.integers(0, mb + 2, n_req) * (g.random(n_req) < 0.8)         # up to one more than the table holds
    n_pages = int(blocks.sum()) + 5
    table = g.integers(-2, n_pages + 3, (n_req, mb)).astype(np.int32)       # absent pages among them
    matched = (blocks * B + g.integers(0, B, n_req)).astype(np.int32)
    matched[g.random(n_req) < 0.05] *= -1
    n_tok = int((np.maximum(matched, 0) // B).sum()) * B
    dev = lambda x: torch.from_numpy(x).to("cuda:0")
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    pools = [dev(g.standard_normal((n_pages, B, hkv, d)).astype(np.float32)).to(t) for _ in "kv"]
    for cut in (0, 37):
        cap = max(n_tok - cut * B, B)
        got = []
        for beside in (False, True):
            ctx = [torch.full((n_tok + B, hkv, d), 7.0, dtype=t, device="cuda:0") for _ in "kv"]
            off = torch.full((n_req + 1,), -7, dtype=torch.int64, device="cuda:0")
            skv.skv_gather_kv(skv.attn_desc(hkv, hkv, d, dtype), *pools, dev(matched), dev(table), mb, off, ctx[0][:cap], ctx[1][:cap],
                              beside=beside)
            got.append([off.cpu()] + [x.cpu() for x in ctx])
        assert all(torch.equal(a, b) for a, b in zip(*got))


def _session(monkeypatch, n_req, least):
    monkeypatch.setattr(pipeline, "GATHER_BESIDE_BYTES", least)
    w = inputs.small_random(seed=n_req, n_seq=8, max_blocks=24, n_req=n_req, vocab=50, attn=inputs.AttnShape(8, 2, 128, "bf16"))
    s = pipeline.Session(w)
    s.prepare()
    return s


def _results(s):
    torch.cuda.synchronize()
    return {k: getattr(s, k).cpu().clone() for k in ("matched_len", "page_table", "q_off", "ctx_off", "out", "kctx", "vctx")}


def _ruin(s):
    for k in ("matched_len", "q_off", "ctx_off", "out", "kctx", "vctx"):
        getattr(s, k).fill_(-7)
    torch.cuda.synchronize()


@pytest.mark.parametrize("n_req", [1, 12, 600])
def test_step_beside_is_the_step(monkeypatch, n_req):
    s = _session(monkeypatch, n_req, 1 << 60)
    _ruin(s)
    s.step()
    want = _results(s)
    s = _session(monkeypatch, n_req, 0)
    assert s.side is not None
    check = lambda: all(torch.equal(a, b) for a, b in zip(want.values(), _results(s).values()))
    for _ in range(3):
        _ruin(s)
        s.step()
        assert check()
    with torch.cuda.stream(torch.cuda.Stream()):
        _ruin(s)
        s.step()
    assert check()
    s.capture_step()
    for _ in range(3):
        _ruin(s)
        s.replay()
        assert check()
        _ruin(s)
        s.step()
        assert check()


def test_attention_refused_leaves_the_copy_joined(monkeypatch):
    s = _session(monkeypatch, 12, 0)
    _ruin(s)
    s.step()
    want = _results(s)
    _ruin(s)
    s.workspace = s.workspace[:64]
    with pytest.raises(skv.SkvError):
        s.step()
    torch.cuda.current_stream().synchronize()     # the copy's stream has joined this one
    assert torch.equal(s.kctx.cpu(), want["kctx"]) and torch.equal(s.ctx_off.cpu(), want["ctx_off"])
