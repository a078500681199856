"""Calls that need no workspace of the context, overlapping on two streams and replayed from a graph beside
direct calls (the surface VJPs of the lumped form, the geometry's VJP).

The reference is the same calls one after the other on a context of their own.  Shared nodes sum at most
a few contributions in another order, over REPS accumulations: 1e-13 relative L2 per call bounds it, the
checks take 1e-12.
"""

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
