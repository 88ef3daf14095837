"""Decode attention where the batch's key tiles are dealt to workgroups in equal shares: requests cut by a share's edge, whole
inside a share, over many shares, empty; more requests than threads; fewer tiles than shares.  Tolerance of the decode tests."""
import numpy as np
import pytest
import torch

from paper_2508_08438_amd import inputs
from test_gpu_decode import check, device_run, oracle_rows

pytestmark = pytest.mark.gpu

G = np.random.default_rng(8)
# contexts, query / kv heads (64 shares of 8 kv heads, 512 of one, 170 of three)
CASES = [
    ([64 * 64], 32, 8), ([64 * 128] * 2, 8, 8), ([64 * 32] * 16, 8, 8),            # edges of shares = edges of requests
    ([0, 0, 64 * 65 + 1, 0, 1, 0], 32, 8), ([30, 0, 2000, 63, 64, 65], 16, 1),     # fewer tiles than shares
    ([20000, 1, 1, 1, 15, 0, 9000], 24, 3), ([1100] + [16] * 300 + [0] * 40 + [1090], 8, 8),
    (G.integers(0, 1300, 700), 4, 1), ([5000] * 3, 6, 6),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_shares(case):
    ctx, hq, hkv = CASES[case]
    dw = inputs.decode_workload(seed=40 + case, ctx=ctx, hard=True, attn=inputs.AttnShape(hq, hkv, 128, "bf16"))
    n = dw.n_req
    check(dw, f"shares {case}", reqs=list(range(n)) if n < 10 else sorted({0, 1, n // 2, n - 2, n - 1, *range(0, n, 61)}))


@pytest.mark.parametrize("n_req,blocks,hkv", [(1, 20, 8), (1, 21, 8), (16, 64, 8), (16, 65, 8)])
def test_both_sides_of_the_rule(n_req, blocks, hkv):
    dw = inputs.decode_workload(seed=n_req + blocks, ctx=[16 * blocks - 3] * n_req, hard=True)
    check(dw, f"{n_req} x {blocks} blocks")


@pytest.mark.parametrize("n_req,hkv,width", [(600, 8, 512), (513, 1, 300), (512, 1, 300), (511, 1, 300), (64, 8, 700), (63, 8, 700)])
def test_wide_tables(n_req, hkv, width):
    # the table says little about the contexts: many requests of a tile or none, some cut, both forms of the list of cut requests
    ctx = np.concatenate([G.choice([0, 0, 1, 16, 63, 64, 65, 130], n_req - 4), [3000, 0, 900, 0]])
    dw = inputs.decode_workload(seed=n_req + hkv, ctx=ctx, hard=True, attn=inputs.AttnShape(2 * hkv, hkv, 128, "bf16"))
    table = np.full((n_req, width), -1, np.int32)
    table[:, : dw.max_blocks] = dw.page_table
    dw.page_table = table
    check(dw, f"wide {n_req}", reqs=sorted({*range(0, n_req, 23), n_req - 4, n_req - 3, n_req - 2, n_req - 1}))


def test_workspace_of_a_larger_batch():
    from paper_2508_08438_amd import binding as skv
    desc = skv.attn_desc(32, 8, 128, "bf16")
    ws = torch.empty(skv.skv_decode_attn_workspace_size(desc, 256, 64), dtype=torch.uint8, device="cuda:0")
    for n_req in (1, 4, 15, 16, 17, 200):
        dw = inputs.decode_workload(seed=n_req, ctx=G.integers(0, 1025, n_req), hard=True)
        table = np.full((n_req, 64), -1, np.int32)
        table[:, : dw.max_blocks] = dw.page_table
        dw.page_table = table
        q, kpool, vpool, want = device_run(dw)
        out = torch.full_like(want, 7.0)
        skv.skv_decode_attn(desc, q, kpool, vpool, torch.from_numpy(dw.ctx_len).to(q.device), torch.from_numpy(table).to(q.device), 64, out, ws)
        assert torch.equal(out, want)


@pytest.mark.parametrize("ctx,hq,hkv", [([32000], 32, 8), ([3000] * 4, 24, 2), ([60, 300, 1000] * 50, 8, 8), ([5000, 77, 900, 12000], 16, 1)])
def test_only_the_output_is_rounded_to_bf16(ctx, hq, hkv):
    # half a unit in the last of the result's eight significant bits: 2^-8 of it.  Weights are right to 2^-16, exponents, whose
    # arguments stay below 128, to 2^-17: together below 2^-15 of the largest value.  (Weights of eight bits: 2^-8 of it.)
    dw = inputs.decode_workload(seed=len(ctx), ctx=ctx, hard=True, attn=inputs.AttnShape(hq, hkv, 128, "bf16"))
    reqs = list(range(len(ctx)))[:6]
    q, kpool, vpool, out = device_run(dw)
    reqs, _, want = oracle_rows(dw, q, reqs)
    got = out[reqs].double().cpu().numpy().reshape(want.shape)
    v_max = float(vpool[~vpool.isnan()].abs().max())
    over = (np.abs(got - want) - np.abs(want) * 2.0 ** -8 * 1.001).max() / v_max
    assert over <= 2.0 ** -15
