"""The current stream's address where torch has no lookup without a Stream object (host-only; the binding looks the names up when
it is imported, so in a process of its own)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import torch
for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
from paper_2404_19124_amd import binding

class Stream:
    cuda_stream = 4711

torch.cuda.is_initialized = lambda: True
torch.cuda.current_stream = lambda: Stream
assert binding._stream_ptr(None) == 4711
"""


def test_current_stream_without_the_raw_lookup():
    run = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr
