"""The binding on a torch that lacks the private raw-stream call: it imports, and what needs no GPU works."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import types
import torch
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream
from paper_2501_02573_amd import binding as b
assert b.query_plan(4, 16, 4096, 128, b.LEET_BF16)[0] >= 1
assert b.workspace_bytes(1, 32, 32768, 128, b.LEET_BF16) > 0
# the handle then comes from the public call
torch.cuda.current_stream = lambda device: types.SimpleNamespace(cuda_stream=1000 + device)
assert b._raw_stream(3) == 1003
"""


def test_import_and_host_queries_without_the_private_stream_call():
    res = subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
