"""The rest of an fp32 step in the attention's launch (up to 64 requests; not where single rows or one-wavefront items run): every output the
same as that of the three stages, in each of the attention's forms and on both sides of the limit."""
import pytest

from test_gpu_step_call import _buffers, _same, _stages, _step

pytestmark = pytest.mark.gpu

CASES = [
    # (query heads, kv heads, d, rows, blocks): eight wavefronts to an item, four; d 128; tiles of 128 rows, 64 requests and 65
    (8, 8, 64, [100, 7], [40, 3]), (8, 4, 64, [33] * 40, [3] * 40), (8, 2, 128, [64, 0, 130], [30, 5, 1]),
    (8, 8, 64, [100, 0, 129] * 21 + [64], [2, 9, 0] * 21 + [1]), (8, 8, 64, [100, 60, 129] * 21 + [64, 1], [2, 9, 0] * 21 + [1, 3]),
    # one wavefront to an item and single rows: launches of their own
    (32, 4, 64, [33, 1] * 32, [2, 1] * 32), (32, 8, 64, [1] * 64, [4] * 64),
    # nothing cached; a copy of 52 MB a pool
    (8, 8, 64, [200, 300], [0, 0]), (16, 16, 64, [20, 40], [300, 530]),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_step_is_its_stages(case):
    hq, hkv, d, S, k = CASES[case]
    desc, c, ws, outputs = _buffers(case + 50, S, k, hq, hkv, d, "f32", max(k) + 1)
    want, got = outputs(), outputs()
    _stages(desc, c, ws, want)
    _step(desc, c, ws, got)
    _same(want, got)
