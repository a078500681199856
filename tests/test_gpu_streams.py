"""Calls that need no workspace of the context, overlapping on two streams and replayed from a graph beside
direct calls (the surface VJPs of the lumped form, the geometry's VJP, the apply on slices).

The VJPs' reference is the same calls one after the other on a context of their own.  Shared nodes sum at most
a few contributions in another order, over REPS accumulations: 1e-13 relative L2 per call bounds it, the
checks take 1e-12.  A slice's node has two columns, so its applies are equal bit by bit.
"""

import ctypes as C

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2506_09435_amd import fnpf
from workloads import configs

REPS = 20
WORKLOADS = {
    "bar": lambda: configs.c4(nx=32, ny=8, nz=4, p=5),
    "box_p8": lambda: configs.small_box(nx=5, ny=4, nz=3, p=8),
    "slice": lambda: configs.small_slice(nx=200, nz=3, p=4),
}


def inputs(s, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda n: torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    return dict(w=r(s.ctx.n_s), ke=r(s.ctx.n_s), kp=r(s.ctx.n_s), lam=r(s.ctx.n_v), phi=r(s.ctx.n_v),
                bars=[torch.zeros(s.ctx.n_s, dtype=torch.float64, device="cuda") for _ in range(5)])


def vjps(s, d):
    e, p, w, h, e2 = d["bars"]
    s.ctx.rhs_vjp(s.eta0, s.phi0, d["w"], d["ke"], d["kp"], e, p, w)
    s.ctx.geom_vjp(d["lam"], d["phi"], e2, h)


def reference(wl, seed, reps):
    s = fnpf.setup_workload(wl)
    s.ctx.geom(s.eta0, s.h)
    d = inputs(s, seed)
    for _ in range(reps):
        vjps(s, d)
    torch.cuda.synchronize()
    return d["bars"]


def close(got, ref):
    return all(float((a - b).norm()) <= 1e-12 * float(b.norm()) for a, b in zip(got, ref))


@pytest.mark.parametrize("name", list(WORKLOADS))
def test_overlapping_vjps(name):
    wl = WORKLOADS[name]()
    ref = [reference(wl, k, REPS) for k in range(2)]
    s = fnpf.setup_workload(wl)
    s.ctx.geom(s.eta0, s.h)
    d = [inputs(s, k) for k in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(REPS):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                vjps(s, d[k])
    torch.cuda.synchronize()
    assert close(d[0]["bars"], ref[0]) and close(d[1]["bars"], ref[1])


@pytest.mark.parametrize("name", list(WORKLOADS))
@pytest.mark.parametrize("same", [False, True])
def test_captured_vjps_beside_direct_ones(name, same):
    wl = WORKLOADS[name]()
    ref = [reference(wl, k, 1) for k in range(2)]
    s = fnpf.setup_workload(wl)
    s.ctx.geom(s.eta0, s.h)
    d = [inputs(s, k) for k in range(2)]
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        vjps(s, d[0])          # a is the context's first stream
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=a if same else b):
        vjps(s, d[1])
    for _ in range(4):
        for x in d[0]["bars"] + d[1]["bars"]:
            x.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(b):
            graph.replay()
        with torch.cuda.stream(a):
            vjps(s, d[0])
        torch.cuda.synchronize()
        assert close(d[0]["bars"], ref[0]) and close(d[1]["bars"], ref[1])


SLICES = [(200, 3, 4), (90, 7, 2), (130, 4, 1), (60, 5, 8), (300, 2, 5)]


def apply_noalloc(ctx, x, y):
    dt = fnpf.F64 if x.dtype == torch.float64 else fnpf.F32
    assert fnpf.lib().fnpf_laplace_apply_noalloc(ctx._h, dt, C.c_void_p(x.data_ptr()), C.c_void_p(y.data_ptr()), 0,
                                                 C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0


@pytest.mark.parametrize("nx,nz,p", SLICES)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_slice_applies_overlap(nx, nz, p, dtype):
    # layers in one block and split, several tiles; both forms of the call, on the context's first stream,
    # on another one beside it and beside a solve, and from a graph: bitwise the same
    wl = configs.small_slice(nx=nx, nz=nz, p=p)
    s = fnpf.setup_workload(wl, fp32=True)
    s.ctx.geom(s.eta0, s.h)
    g = torch.Generator(device="cuda").manual_seed(p)
    x = [torch.randn(s.ctx.n_v, dtype=torch.float64, device="cuda", generator=g).to(dtype) for _ in range(2)]
    ref = [s.ctx.laplace_apply(v) for v in x]      # the default stream is the first
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    y = [torch.full_like(v, float("nan")) for v in x]
    z = torch.full_like(x[0], float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        apply_noalloc(s.ctx, x[1], z)
    for _ in range(REPS):
        with torch.cuda.stream(other):
            s.ctx.laplace_apply(x[1], y[1])
        apply_noalloc(s.ctx, x[0], y[0])
        with torch.cuda.stream(other):
            graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(y[0], ref[0]) and torch.equal(y[1], ref[1]) and torch.equal(z, ref[1])
    phi, info = s.ctx.solve(s.phi0, opts=fnpf.default_opts(rtol=1e-11))
    with torch.cuda.stream(other):
        for _ in range(REPS):
            s.ctx.laplace_apply(x[1], y[1])
    phi2, _ = s.ctx.solve(s.phi0, opts=fnpf.default_opts(rtol=1e-11))
    torch.cuda.synchronize()
    assert info["status"] == "OK" and torch.equal(phi, phi2) and torch.equal(y[1], ref[1])
