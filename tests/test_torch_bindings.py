"""The allocator hook and the current stream on a torch whose private bindings have
other names: the public functions serve."""

import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

CODE = """
import torch
for n in ("_cuda_cudaCachingAllocator_raw_alloc", "_cuda_cudaCachingAllocator_raw_delete",
          "_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, n):
        delattr(torch._C, n)
calls = []
torch.cuda.caching_allocator_alloc = lambda size, device=None, stream=None: calls.append((size, stream)) or 4096
torch.cuda.caching_allocator_delete = lambda ptr: calls.append(ptr)
class Stream:
    cuda_stream = 48
torch.cuda.current_stream = lambda device=None: Stream
import paper_2206_03380_amd as M
assert M._torch_alloc(None, 256, 16) == 4096
M._torch_free(None, 4096, 16)
assert calls == [(256, 16), 4096], calls
assert M._stream().value == 48
print("ok")
"""


def test_public_functions():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-2000:]
