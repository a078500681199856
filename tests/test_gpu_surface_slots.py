"""The surface kernels that leave contributions in face slots (RHS, RHS VJP, geometry VJP) and the
layer groups of the geometry VJP: layer counts that do not divide into the groups and exceed the column
places of a block, every column alone in its block or several, nodes of more than four columns.

Tolerances: the RHS at 1e-12 relative L2 (two rounding-level sums a node).  The VJPs by the identity
<ybar, dF[v]> = <F^T ybar, v> with complex-step dF of the oracle, to 1e-11 of sum |F^T ybar| |v|: each
term passes two derivative matrices (entries to p^2), so rounding stays below 2e-16 p^4 = 1e-12 of it.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import geometry as geo
from oracle import operator as op
from oracle import surface as sf
from paper_2506_09435_amd import fnpf
from workloads import mesh as wm

EPS = 1e-30
MESHES = {
    "box_p8_nz5": lambda: wm.structured_box(2, 2, 0.0, 2.0, 0.0, 1.5, False, False, p=8, nz=5),   # 3 places, 5 layers
    "box_p5_nz4": lambda: wm.structured_box(3, 2, 0.0, 2.0, 0.0, 1.5, True, False, p=5, nz=4),    # 7 places, 4 groups
    "box_p1_nz3": lambda: wm.structured_box(5, 4, 0.0, 2.0, 0.0, 1.5, False, False, p=1, nz=3),
    "box_p2_nz1": lambda: wm.structured_box(3, 3, 0.0, 2.0, 0.0, 1.5, False, True, p=2, nz=1),
    "slice_p8_nz7": lambda: wm.structured_slice(4, 0.0, 2.0, False, p=8, nz=7),
    "slice_p1_nz2": lambda: wm.structured_slice(9, 0.0, 2.0, True, p=1, nz=2),
    "tank": lambda: wm.cylinder_tank_mesh(p=2, nz=3, n_theta=8, n_rad=2, tank=(6.0, 4.0), spacing=1.0, hole_half=1.0),
}


def dev(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def host(t):
    return t.cpu().numpy()


@pytest.mark.parametrize("name", list(MESHES))
def test_surface_kernels_with_slots(name):
    m = MESHES[name]()
    xh = geo.horizontal_coords(m)
    x, y = geo.node_xy(m)
    rng = np.random.default_rng(5)
    eta = 0.05 * np.cos(1.3 * x + 0.2) * np.cos(0.9 * y) + 0.002 * rng.standard_normal(m.n_s)
    phis = 0.1 * np.sin(1.1 * x + 0.7 * y)
    h = 1.0 + 0.1 * np.sin(0.8 * x) + 0.05 * np.cos(y)
    w = 0.2 * np.cos(0.8 * x - 0.4 * y)
    ctx = fnpf.Context(m, g=9.81)
    ke, kp = sf.free_surface_rhs(m, eta, phis, w, 9.81, xh=xh)
    ge, gp = ctx.rhs(dev(eta), dev(phis), dev(w))
    for g, k in ((ge, ke), (gp, kp)):
        assert np.linalg.norm(host(g) - k) <= 1e-12 * np.linalg.norm(k)

    def zeros(n=m.n_s):
        return torch.zeros(n, dtype=torch.float64, device="cuda")

    def check(lhs, bars, vs):
        rhs = sum(host(b) @ v for b, v in zip(bars, vs))
        assert abs(lhs - rhs) <= 1e-11 * sum(np.abs(host(b)) @ np.abs(v) for b, v in zip(bars, vs))

    ve, vp, vw, kbe, kbp = (rng.standard_normal(m.n_s) for _ in range(5))
    de, dp = sf.free_surface_rhs(m, eta + 1j * EPS * ve, phis + 1j * EPS * vp, w + 1j * EPS * vw, 9.81, xh=xh)
    bars = [zeros(), zeros(), zeros()]
    ctx.rhs_vjp(dev(eta), dev(phis), dev(w), dev(kbe), dev(kbp), *bars)
    check(kbe @ (de.imag / EPS) + kbp @ (dp.imag / EPS), bars, (ve, vp, vw))

    lam, phi = rng.standard_normal(m.n_v), rng.standard_normal(m.n_v)
    vh = rng.standard_normal(m.n_s)
    G, _, _ = geo.factors(m, eta + 1j * EPS * ve, h + 1j * EPS * vh, xh)
    A = op.assemble_dense(m, G)
    ctx.geom(dev(eta), dev(h))
    bars = [zeros(), zeros()]
    ctx.geom_vjp(dev(lam), dev(phi), *bars)
    check(-lam @ (A.imag / EPS) @ phi, bars, (ve, vh))
