"""The binding imports, and finds the current stream, on a torch without the
private call that returns a stream's raw handle."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import torch
if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    del torch._C._cuda_getCurrentRawStream
import paper_2509_24416_amd as clq

class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle

seen = []
torch.cuda.current_device = lambda: 3
torch.cuda.current_stream = lambda device=None: (seen.append(device), Stream(77))[1]
assert clq._stream(None) == 77 and seen == [3]
assert clq._stream(Stream(5)) == 5
print("ok")
"""


def test_import_without_the_raw_stream_call():
    r = subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-2000:]
