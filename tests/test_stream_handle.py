"""The binding finds the current stream's handle with torch's public functions
alone, where the private ones that it prefers are missing."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
import sys, types
import torch
if hasattr(torch._C, sys.argv[1]):
    delattr(torch._C, sys.argv[1])
from paper_2505_06703_amd import hs
torch.cuda.is_initialized = lambda: True
torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=7)
assert hs._stream() == 7
assert hs._stream(types.SimpleNamespace(cuda_stream=9)) == 9
"""


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_private_function(missing):
    subprocess.run([sys.executable, "-c", PROGRAM, missing], cwd=ROOT, check=True, timeout=300)
