"""The step behind the lookup as one call, against its three stages called one after the other: every output the same, on both sides of
the limits between its forms (offsets made by the attention's workgroups, by the copy's first one, by a kernel of their own)."""
import numpy as np
import pytest
import torch

from paper_2508_08438_amd import binding as skv

pytestmark = pytest.mark.gpu
B, DEV = 16, "cuda:0"


def _buffers(seed, S, k, hq, hkv, d, dtype, mb):
    g = np.random.default_rng(seed)
    n, T, ctx, t = len(S), int(sum(S)), int(sum(k)) * B, torch.bfloat16 if dtype == "bf16" else torch.float32
    n_pages = int(sum(k)) + 3
    table = np.full((n, mb), -1, np.int32)
    table[np.arange(mb)[None, :] < np.asarray(k, int).reshape(n, 1)] = g.permutation(n_pages)[: int(sum(k))]
    if sum(k) > 4:
        table[int(np.argmax(k)), 1] = n_pages + 2                       # an absent page
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    r = lambda *s: dev(g.standard_normal(s).astype(np.float32)).to(t)
    matched = np.asarray(k, np.int32) * B
    tokens = matched + np.asarray(S, np.int32)
    c = dict(req_off=dev(np.concatenate([[0], np.cumsum(tokens)]).astype(np.int32)), matched=dev(matched), table=dev(table), mb=mb,
             q=r(T, hq, d), knew=r(T, hkv, d), vnew=r(T, hkv, d), kpool=r(n_pages, B, hkv, d), vpool=r(n_pages, B, hkv, d))
    desc = skv.attn_desc(hq, hkv, d, dtype)
    ws = torch.empty(skv.skv_prefill_attn_workspace_size(desc, n, T), dtype=torch.uint8, device=DEV)

    def outputs():
        f = lambda *s, dt=t: torch.full(s, -7, dtype=dt, device=DEV)
        return dict(q_off=f(n + 1, dt=torch.int32), ctx_off=f(n + 1, dt=torch.int64), out=f(T, hq, d), kctx=f(ctx + B, hkv, d), vctx=f(ctx + B, hkv, d))
    return desc, c, ws, outputs


def _step(desc, c, ws, o):
    skv.skv_prefill_step(desc, c["req_off"], c["q"], c["knew"], c["vnew"], o["q_off"], c["kpool"], c["vpool"], c["matched"], c["table"],
                         c["mb"], o["out"], o["ctx_off"], o["kctx"], o["vctx"], ws)


def _stages(desc, c, ws, o, attention=True):
    skv.skv_suffix_offsets(c["req_off"], c["matched"], o["q_off"])
    skv.skv_gather_kv(desc, c["kpool"], c["vpool"], c["matched"], c["table"], c["mb"], o["ctx_off"], o["kctx"], o["vctx"])
    if attention:
        skv.skv_prefill_attn(desc, c["q"], c["knew"], c["vnew"], o["q_off"], c["kpool"], c["vpool"], c["matched"], c["table"], c["mb"],
                             o["out"], ws)


def _same(a, b):
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k].view(torch.uint8).cpu(), b[k].view(torch.uint8).cpu()), k


CASES = [
    # (query heads, kv heads, d, dtype, rows, blocks): split, the offsets in the attention: one request, 30 and 32, rows of none, heads alone;
    (32, 8, 128, "bf16", [137], [187]), (8, 1, 128, "bf16", [1] * 30, [60] * 30), (8, 1, 128, "bf16", [1] * 32, [60] * 32),
    (4, 4, 128, "bf16", [300, 0, 5, 0], [90, 7, 300, 0]), (64, 8, 128, "bf16", [257, 3], [500, 7]), (1, 1, 128, "bf16", [600], [200]),
    # unsplit and with a list: 33, 64, 65 requests; 512 and 513, where the copy no longer scans
    (8, 1, 128, "bf16", [1] * 33, [60] * 33), (8, 2, 128, "bf16", [33, 70] * 32, [1, 9] * 32), (8, 2, 128, "bf16", [33] * 65, [2] * 65),
    (4, 1, 128, "bf16", [3, 0] * 256, [1, 2] * 256), (4, 1, 128, "bf16", [3] * 513, [1] * 513),
    # fp32: the offsets with the copy; a copy of 48 MB a pool, with the fp32 attention and in front of the bf16 one
    (8, 8, 64, "f32", [64, 1, 80], [16, 0, 3]), (4, 2, 64, "f32", [2] * 257, [1] * 257), (8, 8, 128, "f32", [9, 30], [300, 420]),
    (8, 8, 128, "bf16", [40], [1600]),
    # nothing cached, nothing new, nobody
    (8, 2, 128, "bf16", [40], [0]), (8, 2, 128, "bf16", [0, 0], [4, 2]), (8, 2, 128, "bf16", [], []),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_step_is_its_stages(case):
    hq, hkv, d, dtype, S, k = CASES[case]
    desc, c, ws, outputs = _buffers(case, S, k, hq, hkv, d, dtype, max(k, default=0) + 1)
    want, got = outputs(), outputs()
    ws.fill_(0x5a)
    _stages(desc, c, ws, want)
    ws.fill_(0xa5)
    _step(desc, c, ws, got)
    _same(want, got)


@pytest.mark.parametrize("case", [12, 13, 14])
def test_copy_is_the_pages(case):
    """What the stages above are compared with: the copy by torch's indexing, absent pages left as they were."""
    hq, hkv, d, dtype, S, k = CASES[case]
    desc, c, ws, outputs = _buffers(case, S, k, hq, hkv, d, dtype, max(k) + 1)
    want, got = outputs(), outputs()
    _step(desc, c, ws, got)
    pages = torch.cat([c["table"][r, :n] for r, n in enumerate(k)]).long()
    here = (pages >= 0) & (pages < c["kpool"].shape[0])
    for ctx, pool in (("kctx", "kpool"), ("vctx", "vpool")):
        want[ctx][:-B].view(-1, B, hkv, d)[here] = c[pool][pages[here]]
        assert torch.equal(want[ctx], got[ctx])
    assert got["ctx_off"].tolist() == [B * sum(k[:r]) for r in range(len(k) + 1)]


def test_refused_attention_leaves_offsets_and_copy():
    desc, c, ws, outputs = _buffers(1, [137, 20], [40, 3], 32, 8, 128, "bf16", 41)
    want, got = outputs(), outputs()
    _stages(desc, c, ws, want, attention=False)
    with pytest.raises(skv.SkvError):
        _step(desc, c, ws[:64], got)
    _same(want, got)


def test_matched_beyond_the_request_and_short_staging():
    desc, c, ws, outputs = _buffers(2, [137, 20, 5], [40, 3, 2], 32, 8, 128, "bf16", 41)
    c["req_off"] = torch.tensor([0, 777, 797, 812], dtype=torch.int32, device=DEV)     # 777 - 640, max(0, 20 - 48), max(0, 15 - 32)
    want, got = outputs(), outputs()
    for o in (want, got):
        o["kctx"], o["vctx"] = o["kctx"][:B * 21], o["vctx"][:B * 21]
    _stages(desc, c, ws, want)
    _step(desc, c, ws, got)
    _same(want, got)


# counters cleared beside the lookup and updated behind it: 512 requests and 513, which have a launch for each; a split call and fp32
@pytest.mark.parametrize("n_req,dtype,hq,hkv,d", [(1, "bf16", 8, 2, 128), (12, "bf16", 8, 1, 128), (40, "f32", 4, 2, 64), (512, "bf16", 4, 1, 128),
                                                   (513, "bf16", 4, 1, 128)])
def test_counters_of_a_step(n_req, dtype, hq, hkv, d):
    from paper_2508_08438_amd import inputs, pipeline
    w = inputs.small_random(seed=n_req + 5, n_seq=8, max_blocks=24, n_req=n_req, vocab=50, n_tenants=100, attn=inputs.AttnShape(hq, hkv, d, dtype))
    s = pipeline.Session(w)
    s.match()
    want = s.counters()
    assert want[0].sum() > 0
    state = [x.cpu().clone() for x in (s.matched_len, s.page_table, s.q_off)]

    def check():
        assert all(np.array_equal(a, b) for a, b in zip(want, s.counters()))
        assert all(torch.equal(a, b.cpu()) for a, b in zip(state, (s.matched_len, s.page_table, s.q_off)))
    for _ in range(2):
        s.step()
        check()
    s.capture_step()
    for _ in range(3):
        s.replay()
        check()
        s.step()
        check()
    s.workspace = s.workspace[:64]      # an attention that is refused has counted all the same
    with pytest.raises(skv.SkvError):
        s.step()
    check()
