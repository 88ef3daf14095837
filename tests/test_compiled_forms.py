"""The scan of test_compiled_kernels over the kernels' further forms."""
import pytest
from test_compiled_kernels import test_no_early_reader_behind_a_branch as _scan


@pytest.mark.parametrize("src,kernels,need", [
    ("skv_attn_f32.hip", ["attn_f32_kernelILi64ELi8E"], 12),
    ("skv_attn.hip", ["attn_bf16_kernelILb0ELb0ELb0E", "attn_bf16_kernelILb0ELb1ELb0E", "attn_bf16_kernelILb1ELb0ELb0E", "attn_bf16_kernelILb1ELb1ELb0E",
                      "attn_bf16_kernelILb0ELb0ELb1E"], 12),
])
def test_further_forms(src, kernels, need, tmp_path):
    _scan(src, kernels, need, tmp_path)
