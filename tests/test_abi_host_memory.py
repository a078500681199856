"""Mesh headers whose host-side tables cannot be built: fnpf_create returns a status (and a message), it
does not end the process.  Each call runs in a child process, on the CPU: no HIP call is reached."""

import subprocess
import sys
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import sys
sys.path.insert(0, {root!r})
from tests.test_abi import _create
from workloads import mesh as wm
m = wm.structured_box(2, 2, 0.0, 1.0, 0.0, 1.0, False, False, p=2, nz=1)
st, msg, h = _create(m, {over})
assert h.value is None
print(st, msg)
"""


@pytest.mark.parametrize("over,status", [
    ("n_s=1 << 40", 1),       # far more nodes than the elements have: some are unused
    ("n_s=1 << 62", 1),
    ("nz=2**31 - 1", 1),      # the node levels do not fit 32 bits
    ("nz=2**30 - 1", 2),      # 8.6 GB of layer fractions under the limit below
])
def test_create_returns_a_status(over, status):
    limit = "import resource; resource.setrlimit(resource.RLIMIT_AS, (8 << 30, 8 << 30))\n"
    code = CHILD.format(root=ROOT, over=over)
    if status == 2:
        code = code.replace("m = wm", limit + "m = wm")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.returncode, r.stderr[-400:])
    assert r.stdout.startswith(f"{status} ") and len(r.stdout.split(" ", 1)[1].strip()) > 0, r.stdout
