"""Short suffixes of models with eight or sixteen query heads per kv head: both sides of 16 rows, where the host's choice between tiles of
eight heads and of four changes its forecast, whole and split, planned and from a list.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv", [(64, 8), (8, 1), (16, 1)])
@pytest.mark.parametrize("S,k", [([16] * 12, [120] * 12), ([17] * 12, [120] * 12), ([1] * 20, [385] * 20), ([6, 1, 3] * 5, [300, 2, 700] * 5),
                                 ([7, 0, 2, 16] * 18, [35, 3, 0, 20] * 18), ([1] * 79 + [400], [72] * 80), ([15] * 33, [95] * 33)])
def test_short_suffixes(hq, hkv, S, k):
    c = attn_case(sum(S) + hq, len(S), hq, hkv, 128, torch.bfloat16, max(k) + 1, S, k, n_pages=sum(k) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=16)
    assert got.shape == want.shape and np.isfinite(got).all()
    assert np.abs(got - want).max() <= 2e-2
