"""Gather on both sides of the number of requests whose lengths every workgroup scans itself, and of the chunks of the offsets
kernel in front of more: offsets and pages against the oracle, bytes beyond the capacity and of absent pages untouched."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
B = 16


@pytest.mark.parametrize("n_req", [1, 255, 257, 511, 512, 513, 4095, 4096, 4097, 9000])
@pytest.mark.parametrize("cut", [0, 37])
def test_many_requests(n_req, cut):
    from paper_2508_08438_amd import binding as skv
    g = np.random.default_rng(n_req)
    hkv, d, mb = 1, 64, 3
    blocks = g.choice([0, 0, 1, 2, 3], n_req)
    n_pages = int(blocks.sum()) + 5
    table = np.full((n_req, mb), -1, np.int32)
    table[np.arange(mb)[None, :] < blocks[:, None]] = g.permutation(n_pages)[: int(blocks.sum())]
    matched = (blocks * B + g.integers(0, B, n_req)).astype(np.int32)      # whole blocks count
    matched[g.random(n_req) < 0.05] *= -1                                  # and nothing below zero
    blocks = np.maximum(matched, 0) // B
    kpool = torch.from_numpy(g.integers(-30000, 30000, (n_pages, B, hkv, d)).astype(np.int16)).view(torch.bfloat16)
    vpool = torch.from_numpy(g.integers(-30000, 30000, (n_pages, B, hkv, d)).astype(np.int16)).view(torch.bfloat16)
    n_tok = int(blocks.sum()) * B
    cap = max(n_tok - cut * B, B)
    dev = lambda x: (x if torch.is_tensor(x) else torch.from_numpy(x)).to("cuda:0")
    kctx = torch.full((n_tok + B, hkv, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
    vctx = torch.full_like(kctx, 7.0)
    off = torch.full((n_req + 1,), -7, dtype=torch.int64, device="cuda:0")
    gone = g.integers(0, n_req, 4)
    shown = table.copy()
    shown[gone, 0] = [-1, n_pages, n_pages + 9, -5]                        # no such page: those rows stay as they are
    skv.skv_gather_kv(skv.attn_desc(hkv, hkv, d, "bf16"), dev(kpool), dev(vpool), dev(matched), dev(shown), mb, off,
                      kctx[:cap], vctx[:cap])
    want_off = np.concatenate([[0], np.cumsum(blocks * B)])
    assert np.array_equal(off.cpu().numpy(), want_off)
    wk, wv = oracle.gather(kpool, vpool, (blocks * B).astype(np.int32), table)
    for want, got in ((wk, kctx), (wv, vctx)):
        full = torch.full(kctx.shape, 7.0, dtype=torch.bfloat16)
        full[: min(cap, n_tok)] = want[:cap]
        for r in gone:
            if blocks[r] and want_off[r] < cap:
                full[want_off[r]: want_off[r] + B] = 7.0
        assert torch.equal(got.cpu().view(torch.int16), full.view(torch.int16))
