"""A plan's calls in captured graphs: binnings, forwards and adjoints replayed several times,
with new geometries in place and eager calls of the same plan in between, against a fresh
plan of the geometry in use.  (The binning's counters are in two copies of which each binning
clears the other; a graph names one of them for good.)"""
import numpy as np
import pytest

import synth
from gpu_util import torch_gpu

pytestmark = pytest.mark.gpu

LAM, Z0 = 532e-9, 0.1


def _graph(torch, f):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = f()
    torch.cuda.synchronize()
    return g, out


# 32, 1024 and 8192 tiles (the largest in order of size), points over the whole fine grid,
# in part of it (tiles left unwritten) and in a few tiles (compact layout, cut tiles)
@pytest.mark.parametrize("m,p2", [(128, 8e-6), (1024, 8e-6), (2048, 80e-6)])
@pytest.mark.parametrize("first", ["setpts", "forward"])
def test_replays_see_the_binning_before_them(m, p2, first):
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    rng = np.random.default_rng(m)
    n = 30000
    x, y = rng.uniform(-2e-3, 2e-3, n), rng.uniform(-2e-3, 2e-3, n)
    d = synth.sinusoidal_relief(x, y, 20e-6, 0.8e-3)
    x, y, d = (torch.from_numpy(v).cuda() for v in (x, y, d))
    u = torch.from_numpy((rng.uniform(0, 1, n) * np.exp(2j * np.pi * rng.uniform(0, 1, n))).astype(np.complex64)).cuda()
    g2 = torch.from_numpy(synth.random_field(rng, m, m).reshape(m, m)).cuda()
    geo = [x.clone(), y.clone(), d.clone()]
    optics = (LAM, Z0, p2, p2, m, m)

    def place(scale):
        geo[0].copy_(x * scale)
        geo[1].copy_(y * scale)
        fresh = asf.Plan(*geo, *optics)
        want = fresh.forward(u).clone(), fresh.adjoint(g2).clone()
        fresh.close()
        torch.cuda.synchronize()
        return want

    def same(got, want):
        torch.cuda.synchronize()
        return all(torch.equal(torch.view_as_real(a), torch.view_as_real(b)) for a, b in zip(got, want))

    want = place(0.9)
    plan = asf.Plan(*geo, *optics)

    def transforms():
        return plan.forward(u), plan.adjoint(g2)

    def everything():
        plan.setpts(*geo)
        return transforms()

    if first == "setpts":
        bins, got = _graph(torch, everything)
        only, got_only = _graph(torch, transforms)
    else:
        only, got_only = _graph(torch, transforms)
        bins, got = _graph(torch, everything)
    only.replay()
    assert same(got_only, want)
    for scale in (1.0, 1.0, 0.002, 0.3, 1.0, 0.05, 0.002, 1.0):
        want = place(scale)
        bins.replay()
        assert same(got, want), f"replayed binning, scale {scale}"
        assert same(transforms(), want), f"eager transforms after it, scale {scale}"
        only.replay()
        assert same(got_only, want), f"replayed transforms after it, scale {scale}"
    # eager binnings between the replays, and a status read, which may change the binning's path
    for scale in (0.3, 0.002, 0.002, 1.0):
        want = place(scale)
        plan.setpts(*geo)
        assert same(transforms(), want), f"eager binning, scale {scale}"
        only.replay()
        assert same(got_only, want), f"replayed transforms after an eager binning, scale {scale}"
        plan.status()
        bins.replay()
        assert same(got, want), f"replayed binning after an eager one, scale {scale}"
        plan.status()
    plan.close()
