"""Compiled assembly of further matrix-instruction kernels, scanned for readers that come too early behind a branch (see
mfma_hazard_scan).  `need`: idle states a result needs before a vector instruction may read it -- 12 behind the bf16 ones."""
import os
import subprocess

import pytest
from mfma_hazard_scan import scan
from paper_2508_08438_amd import build


@pytest.mark.parametrize("src,kernels,need", [
    ("skv_attn_f32.hip", ["attn_f32_kernelILi64E", "attn_f32_kernelILi128E", "attn_f32_tile_kernel"], 12),
    ("skv_attn_f32.hip", ["attn_f32_kernelILi64ELi1E", "attn_f32_kernelILi64ELi4E", "attn_f32_kernelILi128ELi1E",
                          "attn_f32_kernelILi128ELi4E"], 12),
    ("skv_attn.hip", ["attn_bf16_kernelILb0E", "attn_bf16_kernelILb1E"], 12),
    ("skv_decode.hip", ["decode_attn_kernelILb0E", "decode_attn_kernelILb1E"], 12),
])
def test_no_early_reader_behind_a_branch(src, kernels, need, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    out = str(tmp_path / "k.s")
    r = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", build.INCLUDE, "-I", build.CSRC, "-o", out,
                        os.path.join(build.CSRC, src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    asm = open(out).read()
    for k in kernels:
        assert not scan(asm, k, need=need, horizon=need + 12), k
