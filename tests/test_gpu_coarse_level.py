"""The multigrid's degree-1 level as an assembled operator.  A wrong entry makes the V-cycle another
preconditioner, so CG iteration counts show it: they must be those of the matrix-free level (recorded
with it on the same meshes and data at rtol 1e-11; at most one iteration of slack for rounding).
Covers the one-workgroup form (up to 1,024 unknowns) and the one-launch-a-step form, slices and
boxes, periodic and walled, regular and irregular neighbour counts (the cylinder mesh)."""

import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2506_09435_amd import fnpf
from workloads import configs

MESHES = {
    "box": (lambda: configs.small_box(nx=4, ny=3, nz=2, p=3), 16, 17),
    "wrap": (lambda: configs.small_box(nx=3, ny=3, nz=3, p=4, periodic=(True, True)), 16, 17),
    "walls": (lambda: configs.small_box(nx=21, ny=20, nz=4, p=2, periodic=(False, False), lx=8.0, ly=8.0), 15, 16),
    "tank": (lambda: configs.c3(p=4, nz=2), 87, 99),
    "bar": (lambda: configs.c4(nx=16, ny=4, nz=2, p=5), 49, 52),
    "slice": (lambda: configs.small_slice(nx=5, nz=2, p=4), 16, 17),
    "slice_long": (lambda: configs.small_slice(nx=300, nz=5, p=2, lx=60.0), 16, 17),
    "wave": (lambda: configs.c2(n=12, nz=3, p=6), 16, 17),
}


@pytest.mark.parametrize("name", sorted(MESHES))
def test_assembled_coarse_level(name):
    make, fp64, mixed = MESHES[name]
    s = fnpf.setup_workload(make(), fp32=True)
    x = torch.as_tensor(s.x, device="cuda")
    phis = s.phi0 if name == "wrap" else torch.sin(2 * math.pi * x / float(x.max()))
    for precision, expected in ((0, fp64), (1, mixed)):
        s.ctx.geom(s.eta0, s.h)
        for _ in range(2):
            _, info = s.ctx.solve(phis.contiguous(), opts=fnpf.default_opts(precision=precision, rtol=1e-11,
                                                                           check_every=1))
        assert abs(info["iters"] - expected) <= 1, (precision, info["iters"], expected)
