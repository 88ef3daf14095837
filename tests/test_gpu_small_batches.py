"""Batches that leave compute units idle take forms of their own: pages gathered in slices, fp32 items with eight wavefronts.  Both on
either side of their limits, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_attention_sizes import F32_TOL
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu
B = 16


@pytest.mark.parametrize("pages", [1, 127, 128, 129, 255, 256, 257])                # slots of the table
@pytest.mark.parametrize("hkv,d", [(8, 128), (1, 8), (3, 40), (5, 128)])            # 2048, 16, 240 and 1280 vectors a page
def test_gather_in_slices(pages, hkv, d):
    from paper_2508_08438_amd import binding as skv
    g = np.random.default_rng(pages + d)
    n_req = 1 if pages % 2 else 2
    mb = pages // n_req
    blocks = np.array([mb, mb // 3][:n_req])
    n_pages = int(blocks.sum()) + 2
    table = np.full((n_req, mb), -1, np.int32)
    table[np.arange(mb)[None, :] < blocks[:, None]] = g.permutation(n_pages)[: int(blocks.sum())]
    pools = [torch.from_numpy(g.integers(-30000, 30000, (n_pages, B, hkv, d)).astype(np.int16)).view(torch.bfloat16) for _ in "kv"]
    want = oracle.gather(*pools, (blocks * B).astype(np.int32), table)
    dev = lambda x: (x if torch.is_tensor(x) else torch.from_numpy(x)).to("cuda:0")
    ctx = [torch.full((int(blocks.sum()) * B + B, hkv, d), 7.0, dtype=torch.bfloat16, device="cuda:0") for _ in "kv"]
    off = torch.full((n_req + 1,), -7, dtype=torch.int64, device="cuda:0")
    skv.skv_gather_kv(skv.attn_desc(hkv, hkv, d, "bf16"), dev(pools[0]), dev(pools[1]), dev((blocks * B).astype(np.int32)), dev(table), mb, off, *ctx)
    assert np.array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(blocks * B)]))
    for w, got in zip(want, ctx):
        assert torch.equal(got[:-B].cpu().view(torch.int16), w.view(torch.int16)) and (got[-B:] == 7.0).all()


# (rows / 32 + requests) * heads items: 256 and below eight wavefronts, 264 and above four; keys for none, some and all of them
@pytest.mark.parametrize("hq,hkv", [(8, 8), (8, 2)])
@pytest.mark.parametrize("S,k", [([992], [0]), ([992], [130]), ([1024], [130]), ([64] * 10, [0, 1, 2, 15, 16, 17, 3, 0, 33, 5]),
                                 ([64] * 11, [0, 1, 2, 15, 16, 17, 3, 0, 33, 5, 9]), ([33, 0, 1, 255], [1, 9, 40, 0])])
def test_fp32_few_items(hq, hkv, S, k):
    c = attn_case(sum(S) + hkv, len(S), hq, hkv, 64, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=16)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= F32_TOL
