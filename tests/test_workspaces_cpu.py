"""Workspace sizes: one buffer for the largest batch of a server serves every smaller one."""
import itertools

import pytest

from paper_2508_08438_amd import binding as skv


def never_falls(size, *axes):
    table = {at: size(*(a[i] for a, i in zip(axes, at))) for at in itertools.product(*(range(len(a)) for a in axes))}
    for at, n in table.items():
        for k in range(len(axes)):
            if at[k]:
                less = at[:k] + (at[k] - 1,) + at[k + 1:]
                assert table[less] <= n, ([a[i] for a, i in zip(axes, less)], [a[i] for a, i in zip(axes, at)], table[less], n)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (64, 8), (8, 8), (16, 1), (24, 3), (3, 3)])
def test_decode_workspace_never_falls(hq, hkv):
    desc = skv.attn_desc(hq, hkv, 128, "bf16")
    never_falls(lambda r, b: skv.skv_decode_attn_workspace_size(desc, r, b),
                [0, 1, 2, 3, 8, 15, 16, 17, 64, 127, 128, 129, 256, 511, 512, 1000, 4096], [0, 1, 4, 5, 20, 21, 24, 64, 65, 500, 4096])


@pytest.mark.parametrize("hq,hkv,d,dtype", [(32, 8, 128, "bf16"), (64, 8, 128, "bf16"), (8, 8, 128, "bf16"), (16, 1, 128, "bf16"),
                                            (24, 2, 128, "bf16"), (3, 3, 128, "bf16"), (512, 1, 128, "bf16"), (8, 8, 64, "f32")])
def test_prefill_workspace_never_falls(hq, hkv, d, dtype):
    desc = skv.attn_desc(hq, hkv, d, dtype)
    never_falls(lambda r, n: skv.skv_prefill_attn_workspace_size(desc, r, n),
                [1, 2, 3, 16, 17, 64, 256, 257, 1000, 5000], [0, 1, 31, 32, 33, 64, 137, 500, 2048, 5121, 40000, 1 << 20])
