"""The binding's stream handle and device switch without torch's private short cuts:
a torch that has none takes the public calls (in a process of its own, on the
CPU)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import torch
for owner, names in ((torch._C, ("_cuda_getCurrentRawStream", "_cuda_getDevice")),
                     (torch.cuda, ("_exchange_device", "_maybe_exchange_device"))):
    for n in names:
        if hasattr(owner, n):
            delattr(owner, n)
import paper_1803_08285_amd as sg

class Stream:
    cuda_stream = 4711

entered = []

class Device:
    def __init__(self, d):
        entered.append(d)

torch.cuda.current_stream = lambda *a: Stream()
torch.cuda.device = Device
assert sg._stream() == 4711
t = torch.zeros(1)
assert isinstance(sg._on(t), Device) and entered == [t.device]
print("public calls")
"""


def test_without_the_private_calls():
    r = subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "public calls" in r.stdout, r.stderr[-2000:]
