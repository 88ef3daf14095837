"""The rest of an fp32 step in the attention's launch (up to 64 requests; not where single rows or one-wavefront items run): every output the
same as that of the three stages, in each of the attention's forms and on both sides of the limit."""
import pytest

from test_gpu_f32_tiles import in_tiles
from test_gpu_step_call import _buffers, _same, _stages, _step
from test_gpu_step_rest import launches

pytestmark = pytest.mark.gpu

CASES = [
    # (query heads, kv heads, d, rows, blocks): eight wavefronts to an item, four; d 128; tiles of 128 rows, 64 requests and 65
    (8, 8, 64, [100, 7], [40, 3]), (8, 4, 64, [33] * 40, [3] * 40), (8, 2, 128, [64, 0, 130], [30, 5, 1]),
    (8, 8, 64, [150, 0, 160] * 21 + [64], [2, 17, 0] * 21 + [1]), (8, 8, 64, [120, 60, 129] * 21 + [64, 1], [2, 17, 0] * 21 + [1, 3]),
    # one wavefront to an item and single rows: launches of their own
    (32, 4, 64, [33, 1] * 32, [2, 1] * 32), (32, 8, 64, [1] * 64, [4] * 64),
    # nothing cached; a copy of 52 MB a pool
    (8, 8, 64, [200, 300], [0, 0]), (16, 16, 64, [20, 40], [300, 530]),
    # a large copy, in front: eight wavefronts, small pages; four, few rows
    (4, 2, 64, [1] * 48, [20] * 48), (8, 8, 64, [1] * 60, [7] * 60),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_step_is_its_stages(case):
    hq, hkv, d, S, k = CASES[case]
    assert in_tiles(hq, S, max(k) + 1) == (case in (3, 4))
    desc, c, ws, outputs = _buffers(case + 50, S, k, hq, hkv, d, "f32", max(k) + 1)
    want, got = outputs(), outputs()
    _stages(desc, c, ws, want)
    _step(desc, c, ws, got)
    _same(want, got)


# Either side of the lines of the rule that says so (rest_rides of skv_attn_f32.hip)
@pytest.mark.parametrize("hq,hkv,d,n,rows,blocks,count", [
    # eight wavefronts to an item: 6 MB a pool and 160 items; 48 MB, pages of 16 KB; more than 16 rows, 224 items
    (4, 2, 64, 40, 1, 20, 2), (4, 2, 64, 40, 1, 18, 1), (4, 2, 64, 39, 1, 20, 1), (4, 4, 64, 48, 1, 65, 2), (4, 4, 64, 48, 1, 63, 1),
    (4, 2, 64, 31, 17, 26, 1), (4, 2, 64, 38, 17, 22, 2), (4, 2, 64, 31, 16, 26, 2), (4, 4, 64, 38, 17, 82, 1),
    # four: 12 MB, 440 items, 16 rows
    (8, 8, 64, 60, 1, 7, 2), (8, 8, 64, 60, 1, 6, 1), (8, 8, 64, 54, 1, 10, 1), (8, 8, 64, 55, 1, 10, 2), (8, 8, 64, 40, 17, 10, 1), (8, 8, 64, 40, 16, 10, 2),
    # d 128; a copy of any size in tiles
    (8, 2, 128, 60, 1, 14, 1), (8, 2, 64, 64, 128, 30, 1)])
def test_which_copies_ride(hq, hkv, d, n, rows, blocks, count):
    desc, c, ws, outputs = _buffers(n, [rows] * n, [blocks] * n, hq, hkv, d, "f32", blocks + 1)
    o = outputs()
    assert len(launches(lambda: _step(desc, c, ws, o))) == count
