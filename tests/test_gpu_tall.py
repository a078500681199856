"""A mesh with more layers than a grid has places in y and z (65,536): two columns of 66,000 thin layers, one
iteration with the multigrid.  The iterate is finite and a descent: r.z > 0 would be a breakdown otherwise."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2506_09435_amd import fnpf
from workloads import mesh as wm


def test_more_layers_than_grid_places():
    m = wm.structured_slice(2, 0.0, 1.0, False, p=2, nz=66000)
    ctx = fnpf.Context(m, g=9.81)
    dev = lambda v: torch.full((m.n_s,), v, dtype=torch.float64, device="cuda")
    ctx.geom(dev(0.0), dev(1.0))
    x, _ = ctx.node_xy()
    phi, info = ctx.solve(torch.tensor(x, device="cuda"), raise_on_error=False,
                          opts=fnpf.default_opts(precond=2, rtol=1e-11, max_iter=1, check_every=1))
    assert info["status"] in ("OK", "ERR_NOCONV") and info["iters"] == 1
    assert bool(torch.isfinite(phi).all())
