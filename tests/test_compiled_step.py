"""Compiled assembly of the attention kernels that carry the rest of a step, for which the same holds as without: idle states behind matrix
instructions (mfma_hazard_scan), loads to LDS by scalar descriptors, no spilled register, all forms there."""
import re

import pytest
from mfma_hazard_scan import scan
from test_compiled_loads import FORMS, LOAD, _compile, asm  # noqa: F401


def _scan(text, kernel):   # (nothing runs on behind the end of a program, where the scan would read on: idle states there)
    return scan(text.replace("\ts_endpgm\n", "\ts_endpgm\n\ts_nop 15\n\ts_nop 15\n"), kernel, 12)


def test_forms_are_all_of_them(asm):  # noqa: F811
    assert sorted(re.findall(r"^_ZN\S*attn_rest_kernelI(\w+E)EEv\S*:", asm, re.M)) == sorted(FORMS)


@pytest.mark.parametrize("form", FORMS)
def test_bf16(asm, form):  # noqa: F811
    assert not _scan(asm, "attn_rest_kernelI" + form)
    body = asm[re.search(r"^_ZN\S*attn_rest_kernelI" + form + r"E\S*:", asm, re.M).end():]
    parts = re.split(r"^(\.LBB\w+):", body[:body.index(".Lfunc_end")], flags=re.M)
    blocks = dict(zip(parts[1::2], parts[2::2]))
    assert len(LOAD.findall("".join(parts))) >= 12
    assert not [n for n, b in blocks.items() if LOAD.search(b) and re.search(r"s_cbranch_execnz " + re.escape(n) + r"\b", b)]
    m = re.search(r"\.name:\s+_ZN\S*attn_rest_kernelI" + form + r".*?\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count:\s+(\d+)", asm, re.S)
    assert int(m.group(1)) <= 256 and int(m.group(2)) == 0


F32_STEP = ["attn_f32_tile_kernelILb1E", "attn_f32_kernelILi64ELi4ELb1E", "attn_f32_kernelILi64ELi8ELb1E", "attn_f32_kernelILi128ELi4ELb1E"]


@pytest.fixture(scope="module")
def asm_f32(tmp_path_factory):
    return _compile("skv_attn_f32.hip", tmp_path_factory)


def test_f32(asm_f32):
    for kernel in F32_STEP:
        assert not _scan(asm_f32, kernel)


def test_f32_lengths_are_scanned_in_a_step_only(asm_f32):
    """Where q_off is there already the workgroups don't ask whether it is."""
    kernels = {m.group(1): m.group(2) for m in re.finditer(r"^_ZN\S*?(attn_f32_(?:tile_)?kernelI\w*?Lb[01]E)\S*:(.*?)\.Lfunc_end", asm_f32, re.M | re.S)}
    assert len(kernels) == 2 * len(F32_STEP) + 2 and all(k in kernels for k in F32_STEP)
    for name, body in kernels.items():
        assert ("row_bcast" in body) == (name in F32_STEP), name


@pytest.mark.parametrize("kernel", ["attn_f32_tile_kernelILb0E", "attn_f32_tile_kernelILb1E"])
def test_f32_tiles_spill_outside_their_loop(asm_f32, kernel):
    """The tile kernel holds all 256 registers and spills some: in front of the loop over the blocks of keys and behind it, where that is cheap."""
    body = asm_f32[re.search(r"^_ZN\S*" + kernel + r"\S*:", asm_f32, re.M).end():]
    lines = body[:body.index(".Lfunc_end")].split("\n")
    label = {m.group(1): i for i, x in enumerate(lines) if (m := re.match(r"(\.LBB\w+):", x))}
    back = [(label[m.group(1)], i) for i, x in enumerate(lines) if (m := re.search(r"s_c?branch\S* (\.LBB\w+)", x)) and label[m.group(1)] < i]
    loops = [lines[a:b] for a, b in back if sum("v_mfma" in x for x in lines[a:b]) >= 48]
    assert loops and not [x for loop in loops for x in loop if "scratch_" in x]
