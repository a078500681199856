"""The owner-computes apply with its layers split over several blocks (small meshes), against the
colour schedule of the same library, which assembles in place and splits nothing.

Sizes around the rule (chunks = 1024 blocks / tiles, at most one per layer): one layer per chunk,
ragged chunks (2, 2, 1 and 4, 3 layers), the last split mesh (512 tiles) and the first unsplit one
(513), a ragged last tile.  Both sum the same element contributions in another order: FP64 2e-12
(six contractions of p + 1 <= 9 terms and at most 8 summands per node, condition of the sums <= 1e2
on these meshes), FP32 2e-6, relative 2-norm."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2506_09435_amd import fnpf
from workloads import configs


@pytest.mark.parametrize("p,nx,ny,nz", [(7, 36, 30, 5), (2, 120, 80, 7), (4, 61, 45, 3), (6, 40, 64, 2),
                                        (6, 57, 45, 2), (8, 5, 3, 3), (1, 16, 5, 4)])
def test_split_layers(p, nx, ny, nz):
    wl = configs.c5(nx=nx, ny=ny, nz=nz, p=p)
    s = fnpf.setup_workload(wl, fp32=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(s.ctx.n_v, dtype=torch.float64, device="cuda", generator=g)
    s.ctx.geom(s.eta0, s.h)
    for dt, tol in ((torch.float64, 2e-12), (torch.float32, 2e-6)):
        for mask in (False, True):
            s.ctx.set_apply_variant(0)
            y = s.ctx.laplace_apply(x.to(dt), mask_dirichlet=mask)
            again = s.ctx.laplace_apply(x.to(dt), mask_dirichlet=mask)
            s.ctx.set_apply_variant(7)
            ref = s.ctx.laplace_apply(x.to(dt), mask_dirichlet=mask)
            err = ((y - ref).double().norm() / ref.double().norm()).item()
            assert err < tol, (dt, mask, err)
            assert torch.equal(y, again)


@pytest.mark.parametrize("p,nx,nz", [(4, 8, 2), (4, 120, 3), (4, 20401, 3), (1, 130, 5), (8, 57, 2)])
def test_slice_columns(p, nx, nz):
    """The slices' owner-computes apply (one tile, several, ragged chunks) against the colour
    schedule: same sums, FP64 2e-12 and FP32 2e-6 as above."""
    wl = configs.small_slice(nx=nx, nz=nz, p=p, lx=0.25 * nx)
    s = fnpf.setup_workload(wl, fp32=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(s.ctx.n_v, dtype=torch.float64, device="cuda", generator=g)
    s.ctx.geom(s.eta0, s.h)
    for dt, tol in ((torch.float64, 2e-12), (torch.float32, 2e-6)):
        for mask in (False, True):
            s.ctx.set_apply_variant(0)
            y = s.ctx.laplace_apply(x.to(dt), mask_dirichlet=mask)
            s.ctx.set_apply_variant(7)
            ref = s.ctx.laplace_apply(x.to(dt), mask_dirichlet=mask)
            err = ((y - ref).double().norm() / ref.double().norm()).item()
            assert err < tol, (dt, mask, err)
