"""The bf16 prefill kernel leaves a SIMD 32 vector registers beside its two wavefronts: what gather_beside_kernel runs in."""
import re

import pytest
from test_compiled_loads import FORMS, asm  # noqa: F401


@pytest.mark.parametrize("form", FORMS)
def test_registers(asm, form):  # noqa: F811
    m = re.search(r"\.name:\s+_ZN\S*attn_bf16_kernelI" + form + r".*?\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count:\s+(\d+)", asm, re.S)
    assert (int(m.group(1)) + 7) // 8 * 8 <= 240 and int(m.group(2)) == 0
