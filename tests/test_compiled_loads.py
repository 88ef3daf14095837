"""Compiled assembly.  The bf16 prefill kernel: a load to LDS takes its buffer descriptor from scalar registers.  Where the compiler holds a
part of it in vector registers it wraps the load in a loop over the lanes' values, at the very point where all wavefronts of a workgroup
stand behind a barrier.  The gather of more than 512 requests: offsets and table are read with scalar loads."""
import os
import re
import subprocess

import pytest
from paper_2508_08438_amd import build

LOAD = re.compile(r"buffer_load_dwordx4 .*\blds\b")


def _compile(src, tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    out = str(tmp_path_factory.mktemp("asm") / "k.s")
    r = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", build.INCLUDE, "-I", build.CSRC, "-o", out,
                        os.path.join(build.CSRC, src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return open(out).read()


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    return _compile("skv_attn.hip", tmp_path_factory)


FORMS = ["Lb0ELb0ELb0E", "Lb0ELb1ELb0E", "Lb1ELb0ELb0E", "Lb1ELb1ELb0E", "Lb0ELb0ELb1E"]   # parts, plan, two workgroups


def test_forms_are_all_of_them(asm):
    assert sorted(re.findall(r"^_ZN\S*attn_bf16_kernelI(\w+E)EEv\S*:", asm, re.M)) == sorted(FORMS)


@pytest.mark.parametrize("form", FORMS)
def test_descriptors_are_scalar(asm, form):
    m = re.search(r"^_ZN\S*attn_bf16_kernelI" + form + r"E\S*:", asm, re.M)
    body = asm[m.end():asm.index(".Lfunc_end", m.end())]
    parts = re.split(r"^(\.LBB\w+):", body, flags=re.M)
    blocks = dict(zip(parts[1::2], parts[2::2]))
    assert len(LOAD.findall(body)) >= 12
    looped = [name for name, b in blocks.items() if LOAD.search(b) and re.search(r"s_cbranch_execnz " + re.escape(name) + r"\b", b)]
    assert not looped


def test_gather_reads_offsets_with_scalar_loads(tmp_path_factory):
    asm = _compile("skv_gather.hip", tmp_path_factory)
    m = re.search(r"^_ZN\S*gather_pages_kernelILb0ELb0E\S*:", asm, re.M)
    body = asm[m.end():asm.index(".Lfunc_end", m.end())]
    assert "global_load_dwordx4" in body and not re.search(r"global_load_dword(x2)? ", body)


# A buffer load's range check sets what the lane's offset leaves of the buffer's size *less the scalar offset*: one that lies behind the end
# of a short buffer (a request's last rows, an absent page) is no longer checked against anything.
@pytest.mark.parametrize("kernel", ["attn_f32_tile_kernelILb0E", "attn_f32_tile_kernelILb1E"])
def test_f32_rows_are_in_the_lanes_offset(kernel, tmp_path_factory):
    asm = _compile("skv_attn_f32.hip", tmp_path_factory)
    m = re.search(r"^_ZN\S*" + kernel + r"\S*:", asm, re.M)
    loads = re.findall(r"buffer_load_dword\S* .*", asm[m.end():asm.index(".Lfunc_end", m.end())])
    assert len(loads) >= 30                                              # K and V of the prologue and of either block
    beside = [x for x in loads if not re.match(r"\S+ v\S+, v\d+, s\[\d+:\d+\], 0 offen", x)]
    assert not beside, beside
