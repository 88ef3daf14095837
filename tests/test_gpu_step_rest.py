"""The rest of a bf16 step behind the attention's workgroups, in every form that carries it: every output the same as that of the three
stages, which run the attention without; on both sides of the number of workgroups up to which it does."""
import pytest

from test_gpu_step_call import _buffers, _same, _stages, _step

pytestmark = pytest.mark.gpu

CASES = [
    # (query heads, kv heads, rows, blocks): whole items found in place; from a list; whose longest part is long, split from the list
    (8, 8, [64, 20, 0, 33] * 6, [0, 1, 2, 0] * 6), (32, 8, [100, 300, 0, 129, 64] * 4, [30, 1, 40, 0, 7] * 4), (16, 8, [770, 765, 770], [480, 470, 481]),
    # four wavefronts to a workgroup: 100 requests of up to 17 rows (2024 workgroups), 110
    (32, 8, [17, 16, 9, 17] * 25, [2, 0, 3, 1] * 25), (32, 8, [17, 16] * 55, [2, 3] * 55),
    # eight heads and 32-row tiles; a head alone
    (64, 8, [40, 9, 33, 70] * 8, [10, 40, 3, 0] * 8), (3, 3, [130, 300, 5] * 9, [9, 0, 30] * 9),
    # split in place: long parts, the last request without rows; long items that stay whole, the shortest such table and a shorter one
    (32, 8, [900, 0], [1190, 70]), (64, 8, [118] * 4, [180, 0, 177, 180]), (64, 8, [118] * 4, [71] * 4), (64, 8, [118] * 4, [67, 67, 0, 67]),
    # 512 requests, 513
    (4, 1, [5, 0, 33, 2] * 128, [1, 0, 2, 1] * 128), (4, 1, [5, 0, 33] * 171, [1, 0, 2] * 171),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_step_is_its_stages(case):
    hq, hkv, S, k = CASES[case]
    desc, c, ws, outputs = _buffers(case + 70, S, k, hq, hkv, 128, "bf16", max(k) + 1)
    want, got = outputs(), outputs()
    ws.fill_(0x5a)
    _stages(desc, c, ws, want)
    ws.fill_(0xa5)
    _step(desc, c, ws, got)
    _same(want, got)
