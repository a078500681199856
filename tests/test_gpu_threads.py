"""Contexts of several threads from their first use on: a fresh process in which four threads create a
context each and solve on it at once, on streams of their own.  They run the same kernels on the same data,
so their solutions are equal bit by bit, and equal to a later solve by one thread."""

import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import sys, threading
sys.path.insert(0, {root!r})
import torch
from paper_2506_09435_amd import fnpf
from workloads import configs
wl = configs.small_box(nx=6, ny=5, nz=2, p=6)
torch.zeros(1, device="cuda")
fnpf.lib()
gate, out = threading.Barrier(4), [None] * 4

def solve(k):
    with torch.cuda.stream(torch.cuda.Stream()):
        s = fnpf.setup_workload(wl)
        s.ctx.geom(s.eta0, s.h)
        gate.wait()
        phi, info = s.ctx.solve(s.phi0, opts=fnpf.default_opts(precond=2, rtol=1e-11))
        torch.cuda.current_stream().synchronize()
        return phi.cpu(), info["status"]

def run(k):
    gate.wait()
    out[k] = solve(k)

threads = [threading.Thread(target=run, args=(k,)) for k in range(4)]
for t in threads: t.start()
for t in threads: t.join()
gate = threading.Barrier(1)
ref, _ = solve(0)
assert all(o is not None and o[1] == "OK" and torch.equal(o[0], ref) for o in out), out
print("ok")
"""


def test_first_use_from_threads():
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:] + r.stderr[-2000:]
