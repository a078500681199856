"""Device allocations that fail, one after the other, in every call that allocates on first use: the call
returns an error, the same call succeeds once memory is there, and the context then holds exactly the
allocations of one that never failed (nothing missing, which a later kernel would read through a null
pointer, and nothing lost).  CPU: the library runs on tests/hip_stub.c in child processes."""

import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes as C, json, sys
sys.path.insert(0, {root!r})
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
stub.stub_live_bytes.restype = C.c_size_t
stub.stub_live.restype = stub.stub_failed.restype = C.c_long
stub.stub_fail_at.argtypes = [C.c_long]
import numpy as np
from paper_2506_09435_amd import fnpf
from workloads import mesh as wm
L = fnpf.lib()
dim = {dim}
m = (wm.structured_box(3, 4, 0.0, 2.0, 0.0, 1.5, False, True, p=4, nz=2) if dim == 3 else
     wm.structured_slice(5, 0.0, 2.0, False, p=4, nz=2))
nodes = np.ascontiguousarray(m.eh_nodes, dtype=np.int32)
corner = np.ascontiguousarray(m.eh_corner, dtype=np.float64)
desc = fnpf.MeshDesc(dim=m.dim, p=m.p, nz=m.nz, n_eh=m.n_eh, n_s=m.n_s, eh_nodes=nodes.ctypes.data,
                     eh_corner=corner.ctypes.data, eh_arc=None, eh_face_tag=None, layer_s=None, g=9.81)
surf = [np.ones(m.n_s) for _ in range(8)]
vol = [np.ones(4 * (m.n_v + 2 * m.n_s)) for _ in range(3)]
S = [a.ctypes.data for a in surf]
V = [a.ctypes.data for a in vol]
G = np.zeros(m.n_e * 6 * (m.p + 1) ** 3)
opt = lambda **kw: fnpf.default_opts(rtol=1e-8, **kw)
keep = [opt(), opt(precond=1), opt(precision=1), opt(precision=1, precond=0), opt(line_smoother=1)]
o, jac, mixed, none, line = [C.addressof(x) for x in keep]
geom = lambda h: L.fnpf_geom(h, S[0], S[1], None)
OPS = [
    ("fp32", L.fnpf_enable_fp32),
    ("solve", lambda h: geom(h) or L.fnpf_solve(h, S[2], None, V[0], o, None, None)),
    ("jacobi", lambda h: L.fnpf_solve(h, S[2], None, V[0], jac, None, None)),
    ("mixed", lambda h: geom(h) or L.fnpf_solve(h, S[2], None, V[0], mixed, None, None)),
    ("none", lambda h: L.fnpf_solve(h, S[2], None, V[0], none, None, None)),
    ("line", lambda h: L.fnpf_solve(h, S[2], None, V[0], line, None, None)),
    ("adjoint", lambda h: L.fnpf_solve_adjoint(h, V[0], V[1], jac, None, None)),
    ("filter", lambda h: L.fnpf_set_modal_filter(h, 2, 1.0, 2)),
    ("quadrature", lambda h: L.fnpf_set_surface_quadrature(h, 7)),
    ("relaxation", lambda h: L.fnpf_set_relaxation(h, S[1], S[1], S[1], S[1], S[1], 1.0, 0.0)),
    ("step", lambda h: L.fnpf_rk4_step(h, S[0], S[2], S[1], 0.0, 0.1, jac, V[0], None, None)),
    ("step_vjp", lambda h: L.fnpf_rk4_step_vjp(h, S[1], 0.0, 0.1, V[0], S[3], S[4], S[5], jac, None, None)),
    ("linear", lambda h: L.fnpf_set_linear(h, 1) or L.fnpf_rk4_step(h, S[0], S[2], S[1], 0.0, 0.1, jac, V[0], None, None)),
    ("linear_vjp", lambda h: L.fnpf_rk4_step_vjp(h, S[1], 0.0, 0.1, V[0], S[3], S[4], S[5], jac, None, None)),
    ("export", lambda h: L.fnpf_export_geometry(h, 0, G.ctypes.data, V[1], None)),
    ("stored", lambda h: L.fnpf_set_apply_variant(h, 1) or geom(h)),
]

def create():
    h = C.c_void_p()
    return L.fnpf_create(C.byref(desc), C.byref(h)), h

def live():
    return stub.stub_live(), stub.stub_live_bytes()

def context(first):
    st, h = create()
    assert st == 0, st
    for name, op in OPS[:first]:
        assert op(h) == 0, (name, L.fnpf_last_error(h))
    return h

bad, tried = [], 0
for k in range(1, 1000):      # creation itself
    stub.stub_fail_at(k)
    st, h = create()
    hit = stub.stub_failed()
    stub.stub_fail_at(0)
    if st == 0:
        L.fnpf_destroy(h)
    if not hit:
        break
    tried += 1
    if st == 0 or live() != (0, 0):
        bad.append(("create", k, st, live()))
for i, (name, op) in enumerate(OPS):
    h = context(i + 1)
    want = live()
    L.fnpf_destroy(h)
    if live() != (0, 0):
        bad.append((name, "left after destroy", live()))
    for k in range(1, 1000):
        h = context(i)
        stub.stub_fail_at(k)
        st = op(h)
        hit = stub.stub_failed()
        stub.stub_fail_at(0)
        again = op(h)
        got = live()
        L.fnpf_destroy(h)
        if not hit:
            break
        tried += 1
        if st == 0 or again != 0 or got != want:
            bad.append((name, k, st, again, got, want))
print(json.dumps(dict(bad=bad, tried=tried)))
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no host C compiler")
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-w", os.path.join(ROOT, "tests", "hip_stub.c"), "-o", so], check=True)
    return so


@pytest.mark.parametrize("dim", [2, 3])
def test_failed_allocations(stub, dim):
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, stub=stub, dim=dim)], capture_output=True,
                       text=True, timeout=110)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    out = json.loads(r.stdout.splitlines()[-1])
    assert out["tried"] > 150 and not out["bad"], out["bad"][:20]
