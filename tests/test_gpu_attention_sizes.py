"""Prefill attention at the sizes where its kernels change form: edges of row tiles and key blocks, many and empty
requests, absent pages.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu

# fp32: a softmax weight 2^x carries a relative error of about |x| 2^-23 (the rounding of the exponent's argument, |x| <=
# 40 for these scores), the two sums add less; a weighted mean of values up to 5 is then within 5 * 40 * 2^-23 = 2.4e-5.
F32_TOL = 4e-5


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (4, 2, 64), (2, 2, 128), (8, 2, 128)])
@pytest.mark.parametrize("S,k", [
    ([1], [0]), ([1], [1]), ([31, 32, 33, 1], [0, 2, 1, 3]),     # one block of keys, one tile of rows, one more
    ([127, 128, 129, 0, 97], [0, 0, 8, 3, 7]),                   # keys for one round of the four wavefronts, and one more
    ([300], [20]),
    ([0, 0, 3] + [5, 0, 33] * 43 + [0], [1] * 133),              # more than 64 requests, empty ones among them
])
def test_fp32_tiles_and_key_blocks(hq, hkv, d, S, k):
    c = attn_case(sum(S) + hq + d, len(S), hq, hkv, d, torch.float32, max(k) + 1, S, k, n_pages=sum(k) + 3)
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= F32_TOL


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_absent_pages_read_as_zeros(d):
    c = attn_case(5, 3, 4, 2, d, torch.float32, 9, [1, 20, 70], [1, 5, 9], n_pages=40)
    for r, j in ((0, 0), (1, 1), (1, 4), (2, 0), (2, 8)):
        for pool in ("kpool", "vpool"):
            c[pool][c["page_table"][r, j]] = 0
    want = oracle.attention(**c, n_threads=8)
    for n, (r, j) in enumerate(((0, 0), (1, 1), (1, 4), (2, 0), (2, 8))):
        c["page_table"][r, j] = -1 if n % 2 else 40 + n
    assert np.abs(run_attn(c) - want).max() <= F32_TOL


def test_fp32_maxima_that_keep_moving():
    # scores rising over hundreds of exp2 units along the keys: every block moves the running maximum.  The weights that
    # count lie within a few units of the maximum; their score is rounded at 2^-24 * 400, five of those per exponent.
    c = attn_case(9, 2, 2, 2, 64, torch.float32, 5, [200, 90], [4, 0])
    c["q"][:] = 1.0
    n = c["knew"].shape[0]
    c["knew"][:] = torch.arange(n, dtype=torch.float32)[:, None, None] * 0.05
    c["kpool"][:] = -1.0
    got, want = run_attn(c), oracle.attention(**c, n_threads=8)
    assert np.abs(got - want).max() <= 5 * 5 * 400 * 2.0 ** -24
