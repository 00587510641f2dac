"""The caller's stream handle, with torch's private accessor and without it."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
import types, torch
torch.cuda.current_device = lambda: 2
torch.cuda.current_stream = lambda *a: types.SimpleNamespace(cuda_stream=0x1234)
%s
from paper_2305_04711_amd import cpm
print(hex(cpm._stream().value))
"""


@pytest.mark.parametrize("accessor,handle", [
    ("torch._C._cuda_getCurrentRawStream = lambda d: 0x5678 + d", "0x567a"),
    ("if hasattr(torch._C, '_cuda_getCurrentRawStream'): del torch._C._cuda_getCurrentRawStream",
     "0x1234")])
def test_stream_handle(accessor, handle):
    out = subprocess.run([sys.executable, "-c", PROGRAM % accessor], cwd=ROOT, check=True,
                         capture_output=True, text=True).stdout
    assert out.strip() == handle
