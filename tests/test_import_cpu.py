"""A torch without GPU support, which lacks the functions that the binding reads the current stream with, imports the package (its oracle and
index tests need no GPU)."""
import os
import subprocess
import sys

CODE = """
import torch
for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
torch.cuda.current_stream = lambda: type("S", (), {"cuda_stream": 77})
from paper_2508_08438_amd import binding
assert binding._stream(None) == 77
"""


def test_import_without_gpu_support():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE], cwd=root, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
