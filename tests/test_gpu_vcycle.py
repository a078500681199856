"""One V-cycle of the multigrid preconditioner by value: the first CG iteration from zero is alpha V(b), so
that its iterate holds every value that the cycle leaves at the unknowns.  The reference is the same cycle
in plain FP64 with the oracle's operators and diagonals on every level, interpolation matrices and their
transposes, and the library's own eigenvalue estimates: it checks the restricted residual (by the apply or
by a kernel of its own), the assembled degree-1 rows, the prolongation and the smoothing together.

Tolerances: a cycle is some 30 products of relative rounding p^2 eps (the derivative tables' entries), which
the smoothing does not amplify: 30 * 64 * 1.1e-16 = 2e-13 in FP64 and 30 * 64 * 6e-8 = 1e-4 in FP32.  One wrong
coarse value of n shows as about 1/sqrt(n), above 1e-2.  FP64 takes 1e-11.
"""

import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import geometry as geo
from oracle import operator as op
from oracle.gll import gll, lagrange_eval
from paper_2506_09435_amd import fnpf
from workloads import mesh as wm


def fan(v, rings, p, nz):
    a = np.pi * np.arange(2 * v) / v
    xy = [(0.0, 0.0)] + [(r * np.cos(t), r * np.sin(t)) for r in range(1, rings + 1) for t in a]
    at = lambda r, k: 1 + (r - 1) * 2 * v + k % (2 * v)
    quads = [(0, at(1, 2 * k), at(1, 2 * k + 1), at(1, 2 * k + 2)) for k in range(v)]
    quads += [(at(r, k), at(r + 1, k), at(r + 1, k + 1), at(r, k + 1)) for r in range(1, rings) for k in range(2 * v)]
    return wm.quad_mesh_from_vertices(np.array(xy), np.array(quads), p, nz)


def box(nx, ny, nz, px, py):
    return lambda p: wm.structured_box(nx, ny, 0.0, 0.5 * nx, 0.0, 0.5 * ny, px, py, p=p, nz=nz)


MESHES = {
    # ragged tiles with the layers split over blocks, every degree
    **{f"box_p{p}": (box(*n, False, p % 2 == 0), p) for p, n in
       {2: (7, 5, 5), 3: (6, 5, 3), 4: (5, 3, 3), 5: (5, 3, 4), 6: (4, 3, 3), 7: (3, 3, 2), 8: (3, 3, 2)}.items()},
    "box_one_tile": (box(3, 3, 3, True, True), 4),
    "box_large": (box(24, 21, 2, True, False), 3),              # degree 1: more than 1,024 unknowns
    "fan_5": (lambda p: fan(5, 3, p, 3), 4),                     # rows of 11 entries a level
    "fan_6": (lambda p: fan(6, 9, p, 5), 2),                     # 13, one launch a step
    "fan_7": (lambda p: fan(7, 3, p, 2), 3),                     # 15, the width as an argument
    "slice_p4": (lambda p: wm.structured_slice(300, 0.0, 20.0, True, p=p, nz=3), 4),   # degree 1: the same
    "slice_p8": (lambda p: wm.structured_slice(40, 0.0, 4.0, False, p=p, nz=4), 8),
    "slice_p2_small": (lambda p: wm.structured_slice(9, 0.0, 2.0, False, p=p, nz=2), 2),
}


def interpolation(f, c):
    """Rows: the nodes of mesh f, each from the first element that has it; columns: those of mesh c."""
    ip = lagrange_eval(c.p, gll(f.p)[0])
    loc = np.kron(ip, ip) if f.dim == 2 else np.kron(np.kron(ip, ip), ip)
    df, dc = geo.dof_map(f), geo.dof_map(c)
    dof, first = np.unique(df.ravel(), return_index=True)
    e, t = np.divmod(first, df.shape[1])
    rows = np.repeat(dof, loc.shape[1])
    return sp.csr_matrix((loc[t].ravel(), (rows, dc[e].ravel())), shape=(f.n_v, c.n_v))


def surface_interpolation(f, c):
    """Values at the horizontal nodes of c of the polynomials of f."""
    w = lagrange_eval(f.p, gll(c.p)[0])
    loc = w if f.dim == 2 else np.kron(w, w)
    e, t = np.divmod(np.unique(c.eh_nodes.ravel(), return_index=True)[1], c.nh)
    return lambda u: np.einsum("nk,nk->n", loc[t], u[f.eh_nodes[e]])


class Cycle:
    def __init__(self, make, p, eta, h, lam):
        self.levels = []
        m = make(p)
        while True:
            G, _, _ = geo.factors(m, eta, h, geo.horizontal_coords(m))
            inner = np.arange(m.n_v) < m.n_v - m.n_s
            self.levels.append(dict(m=m, G=G, dofs=geo.dof_map(m), inner=inner,
                                    dinv=inner / op.diagonal(m, G), lam=lam[len(self.levels)]))
            if m.p == 1:
                break
            c = make(m.p // 2)
            P = interpolation(m, c)
            self.levels[-1]["P"] = P
            s = surface_interpolation(m, c)
            H, h = s(eta + h), s(h)
            eta, m = H - h, c

    def product(self, L, x):
        return op.apply(L["m"], L["G"], x, L["dofs"]) * L["inner"]

    def chebyshev(self, L, b, x, steps, ratio):
        hi = 1.1 * L["lam"]
        lo = hi / ratio
        theta, delta = 0.5 * (hi + lo), 0.5 * (hi - lo)
        rho = delta / theta
        r = b - self.product(L, x)
        d = L["dinv"] * r / theta
        x = x + d
        for _ in range(steps - 1):
            r = r - self.product(L, d)
            rho1 = 1.0 / (2.0 * theta / delta - rho)
            d = rho1 * rho * d + 2.0 * rho1 / delta * L["dinv"] * r
            x, rho = x + d, rho1
        return x

    def __call__(self, b, l=0):
        L = self.levels[l]
        if l + 1 == len(self.levels):
            return self.chebyshev(L, b, 0.0 * b, 10, 30.0)
        x = self.chebyshev(L, b, 0.0 * b, 2, 24.0)
        C = self.levels[l + 1]
        x = x + L["inner"] * (L["P"] @ self(C["inner"] * (L["P"].T @ (b - self.product(L, x))), l + 1))
        return self.chebyshev(L, b, x, 2, 24.0)


@pytest.mark.parametrize("name", list(MESHES))
def test_vcycle_values(name):
    make, p = MESHES[name]
    m = make(p)
    x, y = geo.node_xy(m)
    rng = np.random.default_rng(3)
    lx = 2 * np.pi / max(x.max() - x.min(), 1.0)
    eta, h = 0.03 * np.cos(lx * x + 0.3), 1.0 + 0.1 * np.sin(lx * x)
    phis = rng.standard_normal(m.n_s)
    ctx = fnpf.Context(m, g=9.81)
    ctx.enable_fp32()
    dev = lambda u: torch.tensor(u, dtype=torch.float64, device="cuda")
    for precision, variants, tol in ((0, (0, 6), 1e-11), (1, (0,), 1e-4)):
        for variant in variants:
            ctx.set_apply_variant(variant)
            ctx.geom(dev(eta), dev(h))
            phi, info = ctx.solve(dev(phis), raise_on_error=False, opts=fnpf.default_opts(
                precision=precision, precond=2, rtol=1e-14, inner_rtol=1e-6, max_iter=1, check_every=1))
            assert info["status"] == "ERR_NOCONV" and info["iters"] == 1
            cycle = Cycle(make, p, eta, h, ctx.multigrid_info()["lam32" if precision else "lam64"])
            L = cycle.levels[0]
            lift = np.concatenate([np.zeros(m.n_v - m.n_s), phis])
            b = -cycle.product(L, lift)
            z = cycle(b)
            ref = (b @ z) / (z @ cycle.product(L, z)) * z
            got = phi.cpu().numpy() * L["inner"]
            assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref), (precision, variant)
