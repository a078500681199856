"""Mixed-precision solves on a context that has solved in FP64 before its FP32 path was enabled: the
masks of the preconditioners without a Jacobi diagonal then exist in FP64 only.

Both solutions meet rtol 1e-11 on a system of condition below 1e4, so they agree to 1e-7; the steps'
states agree to the same.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2506_09435_amd import fnpf
from workloads import configs


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("precond", [0, 1, 2])
def test_mixed_solve_after_fp64_solve(dim, precond):
    wl = configs.small_box(nx=4, ny=3, nz=2, p=3) if dim == 3 else configs.small_slice(nx=5, nz=2, p=4)
    s = fnpf.setup_workload(wl)
    opts = lambda precision: fnpf.default_opts(precision=precision, precond=precond, rtol=1e-11, inner_rtol=1e-4)
    s.ctx.geom(s.eta0, s.h)
    ref, info = s.ctx.solve(s.phi0, opts=opts(0))
    assert info["status"] == "OK"
    s.ctx.enable_fp32()
    s.ctx.geom(s.eta0, s.h)
    phi, info = s.ctx.solve(s.phi0, opts=opts(1))
    assert info["status"] == "OK"
    assert float((phi - ref).norm()) <= 1e-7 * float(ref.norm())
    # steps enable the path by themselves
    state = []
    for first in (0, 1):
        t = fnpf.setup_workload(wl)
        for precision in (first, 1):
            e, p = t.eta0.clone(), t.phi0.clone()
            t.ctx.rk4_step(e, p, t.h, 0.0, 0.02, opts=opts(precision))
        state.append((e, p))
    for a, b in zip(*state):
        assert float((a - b).norm()) <= 1e-7 * float(b.norm())
