"""The end of a CG solve inside a running kernel: the blocks of a vector kernel form alpha for themselves
while the first of them may set the done flag (CPU check of csrc/reduce.h with one block as host threads),
and a breakdown of p.Ap leaves the solution at its last iterate (GPU)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include"


def test_block_decides_as_one(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(HIP):
        pytest.skip("no host C++ compiler or no HIP headers")
    exe = str(tmp_path / "cg_flag_check")
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", HIP, "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2506_09435_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cg_flag_check.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


@pytest.mark.gpu
def test_breakdown_keeps_the_last_iterate():
    # on a box of centimetres the diagonal is below 1, so with ||r||^2 at 2.5e299 the first z.Az is above
    # the 1e300 that the solve takes for a breakdown
    import torch

    from paper_2506_09435_amd import fnpf
    from workloads import mesh as wm

    m = wm.structured_box(3, 2, 0.0, 0.03, 0.0, 0.02, False, False, p=3, nz=2)
    ctx = fnpf.Context(m, g=9.81)
    dev = lambda v: torch.full((m.n_s,), v, dtype=torch.float64, device="cuda")
    ctx.geom(dev(0.0), dev(0.01))
    x, _ = ctx.node_xy()
    phis = torch.tensor(x, device="cuda") * 100.0
    _, info = ctx.solve(phis, opts=fnpf.default_opts(precond=1, rtol=1e-11))
    phis *= 5e149 / info["bnorm"]
    phi, info = ctx.solve(phis, opts=fnpf.default_opts(precond=1, rtol=1e-11), raise_on_error=False)
    assert info["status"] == "ERR_BREAKDOWN", info
    assert float(phi[:-m.n_s].abs().max()) == 0.0 and torch.equal(phi[-m.n_s:], phis)
