"""fp32 prefill attention is as exact as fp32: against the fp64 oracle, for each of its kernels and over the magnitudes fp32 has.

Bound: a weight 2^x carries |x| 2^-24 from the rounding of its exponent's argument (|x| about 8 for the keys that count), its
score and the sums less; as a 2-norm over results these are independent, and 8 * 2^-24 = 4.8e-7 is not reached.  With two bf16
pieces instead of three the products are off by 2^-17 and the results by 2e-6 to 7e-6."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import attn_case, run_attn

pytestmark = pytest.mark.gpu
REL = 8 * 2.0 ** -24

G = np.random.default_rng(5)
MANY = dict(S=G.choice([1, 2, 3, 33, 40], 600, p=[.5, .3, .1, .05, .05]), k=G.choice([0, 1, 2, 3, 9], 600))
# query / kv heads, head size, rows and reused blocks per request
CASES = {
    "four wavefronts": (4, 2, 64, [40, 130, 7], [10, 30, 64]),
    "four wavefronts, 128": (8, 2, 128, [40, 130, 7], [10, 30, 64]),
    "one wavefront": (8, 4, 64, MANY["S"], MANY["k"]),
    "one wavefront, 128": (8, 2, 128, MANY["S"][:300], MANY["k"][:300]),
    "rows": (8, 4, 64, [1] * 300, MANY["k"][:300]),
    "rows, 128": (8, 2, 128, [1] * 300 + [2] * 20 + [0] * 5, [*MANY["k"][:324], 70]),
    "128 rows": (16, 2, 64, [257, 383, 384, 385, 511, 512, 513, 130, 1000, 640], [0, 1, 2, 3, 4, 5, 0, 70, 9, 33]),
}


def case(name, seed=1):
    hq, hkv, d, S, k = CASES[name]
    return attn_case(seed, len(S), hq, hkv, d, torch.float32, max(k) + 1, S, k, n_pages=int(sum(k)) + 3)


def compare(c, want):
    got = run_attn(c)
    assert np.isfinite(got).all()
    assert np.linalg.norm(got - want) <= REL * np.linalg.norm(want)
    return got


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("spread", [1.0, 4.0])
def test_as_exact_as_fp32(name, spread):
    c = case(name)
    c["q"] *= spread
    compare(c, oracle.attention(**c, n_threads=16))


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("q,k,v", [(0, 0, -118), (118, -118, 0), (-118, 118, 0), (60, -60, 60), (0, 0, 100)])
def test_magnitudes(name, q, k, v):
    # powers of two change nothing but exponents: the results are those of the same case without them, times 2^v
    c = case(name)
    want = oracle.attention(**c, n_threads=16)
    c["q"] *= 2.0 ** q
    for n, e in (("knew", k), ("kpool", k), ("vnew", v), ("vpool", v)):
        c[n] *= 2.0 ** e
    compare(c, want * 2.0 ** v)


@pytest.mark.parametrize("name", CASES)
def test_small_and_zero_columns(name):
    c = case(name)
    for n in ("vnew", "vpool"):
        c[n][..., 5] *= 2.0 ** -118
        c[n][..., 9] = 0.0
    want = oracle.attention(**c, n_threads=16)
    got = compare(c, want)
    assert np.linalg.norm(got[..., 5] - want[..., 5]) <= REL * np.linalg.norm(want[..., 5])
    assert not got[..., 9].any()


@pytest.mark.parametrize("name", ["one wavefront", "one wavefront, 128"])
def test_values_without_pieces(name):
    # what is not finite reaches the rows that see it and no others
    c = case(name)
    want = oracle.attention(**c, n_threads=16)
    r = int(np.flatnonzero((np.asarray(CASES[name][3]) == 33) & (np.asarray(CASES[name][4]) > 0))[0])
    first = int(c["q_off"][r])
    c["vnew"][first + 20, 0, 3] = float("inf")
    c["knew"][first + 30] = float("nan")
    got = run_attn(c)
    G = c["q"].shape[1] // c["knew"].shape[1]
    seen = np.zeros(got.shape, bool)
    seen[first + 20: first + 33, :G, 3] = True
    seen[first + 30: first + 33] = True
    assert np.linalg.norm((got - want)[~seen]) <= REL * np.linalg.norm(want[~seen])
    assert np.isposinf(got[first + 20: first + 30, :G, 3]).all() and np.isnan(got[first + 30: first + 33]).all()
