"""The package imports, and finds the current stream, on a torch without the private lookups that
it uses to do so faster."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("gone", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_import_without_private_stream_lookup(gone):
    code = f"""
import torch
if hasattr(torch._C, "{gone}"):
    del torch._C.{gone}
import paper_0710_0066_amd as sap

class Stream:
    cuda_stream = 4711

torch.cuda.current_stream = lambda *a: Stream()
assert sap._stream() == 4711
"""
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
