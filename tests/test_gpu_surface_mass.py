"""The surface mass product and its Chebyshev solve at the edges of the line kernel's range: every
degree with the fewest and the most quadrature points (lines shorter and longer than a column's node
rows, one to many columns a block) and column counts that leave a block ragged.

Tolerance: 1e-12 relative L2 against the oracle's dense solve: the iteration's length is set for a
1e-15 contraction, and the quadrature sums some thousand terms.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import geometry as geo
from oracle import surface as sf
from paper_2506_09435_amd import fnpf
from workloads import mesh as wm


def rel(a, b):
    return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)


@pytest.mark.parametrize("nq", [0, 24])
@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("dim", [2, 3])
def test_consistent_rhs_every_degree(dim, p, nq):
    if dim == 3:
        m = wm.structured_box(4 if p < 5 else 3, 3 if p < 5 else 2, 0.0, 2.0, 0.0, 1.5, False, p < 5, p=p, nz=1)
    else:
        m = wm.structured_slice(133 if p < 3 else 5, 0.0, 4.0, p % 2 == 0, p=p, nz=1)
    nq = nq or p + 1
    x, y = geo.node_xy(m)
    rng = np.random.default_rng(p)
    eta = 0.05 * np.cos(1.3 * x + 0.2) * np.cos(0.9 * y) + 0.002 * rng.standard_normal(m.n_s)
    phi = 0.1 * np.sin(1.1 * x + 0.7 * y) + 0.002 * rng.standard_normal(m.n_s)
    w = 0.2 * np.cos(0.8 * x - 0.4 * y) + 0.002 * rng.standard_normal(m.n_s)
    ctx = fnpf.Context(m, g=9.81)
    ctx.set_surface_quadrature(nq)
    ke, kd = sf.free_surface_rhs_consistent(m, eta, phi, w, 9.81, nq)
    ge, gd = ctx.rhs(*(torch.tensor(a, device="cuda") for a in (eta, phi, w)))
    assert rel(ge, ke) < 1e-12 and rel(gd, kd) < 1e-12
