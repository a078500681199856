"""VJP of the consistent surface right-hand side at the highest degrees, where an element has more nodes
than the threads it gets (degree 8: 81 nodes; 64 threads at nq = 9 .. 11, where four elements share a
block, 128 or 256 beyond), with blocks left ragged.

<kbar, dF[v]> = <F^T kbar, v> with complex-step dF of the oracle, to 1e-11 of sum |F^T kbar| |v|: a term
passes two derivative tables (entries to p^2) and a mass solve of condition 5 contracted to 1e-15, so
rounding stays below 2e-16 p^4 = 1e-12 of it.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import geometry as geo
from oracle import surface as sf
from paper_2506_09435_amd import fnpf
from workloads import mesh as wm

EPS = 1e-30


@pytest.mark.parametrize("p,nq", [(8, 9), (8, 10), (8, 11), (8, 12), (8, 24), (7, 8), (7, 24)])
def test_consistent_rhs_vjp_high_degree(p, nq):
    m = wm.structured_box(3, 2, 0.0, 2.0, 0.0, 1.5, False, False, p=p, nz=1)
    x, y = geo.node_xy(m)
    rng = np.random.default_rng(nq)
    eta = 0.05 * np.cos(1.3 * x + 0.2) * np.cos(0.9 * y) + 0.002 * rng.standard_normal(m.n_s)
    phi = 0.1 * np.sin(1.1 * x + 0.7 * y)
    w = 0.2 * np.cos(0.8 * x - 0.4 * y)
    ve, vp, vw, kbe, kbp = (rng.standard_normal(m.n_s) for _ in range(5))
    ke, kd = sf.free_surface_rhs_consistent(m, eta + 1j * EPS * ve, phi + 1j * EPS * vp, w + 1j * EPS * vw, 9.81, nq)
    lhs = kbe @ (ke.imag / EPS) + kbp @ (kd.imag / EPS)
    ctx = fnpf.Context(m, g=9.81)
    ctx.set_surface_quadrature(nq)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    bars = [torch.zeros(m.n_s, dtype=torch.float64, device="cuda") for _ in range(3)]
    ctx.rhs_vjp(dev(eta), dev(phi), dev(w), dev(kbe), dev(kbp), *bars)
    bars = [b.cpu().numpy() for b in bars]
    rhs = sum(b @ v for b, v in zip(bars, (ve, vp, vw)))
    assert abs(lhs - rhs) <= 1e-11 * sum(np.abs(b) @ np.abs(v) for b, v in zip(bars, (ve, vp, vw)))
