"""skv_mfma_rate measures the matrix instruction that the bf16 prefill kernel issues, and no other."""
import re

from test_compiled_loads import asm  # noqa: F401


def test_the_rate_is_of_the_attention_instruction(asm):  # noqa: F811
    used = {}
    for m in re.finditer(r"^(_ZN\S*(?:mfma_rate_kernel|attn_bf16_kernel)\S*):", asm, re.M):
        body = asm[m.end():asm.index(".Lfunc_end", m.end())]
        used[m.group(1)] = set(re.findall(r"\bv_mfma_\w+", body))
    assert len(used) == 7 and all(v == {"v_mfma_f32_16x16x32_bf16"} for v in used.values()), used
