"""GPU parity of the one-dimensional (line) path against the FP64 oracle's 1D
form of Eq. (7): the paper's two profiles (Sec. 3), ragged and wrapping
inputs, a single point, clustered points, the largest sizes, batches and
bitwise repeatability."""
import os

import numpy as np
import pytest

import synth
from gpu_util import rel_l2, torch_gpu

pytestmark = pytest.mark.gpu

TOL = 1e-5
ORACLE_THREADS = min(16, os.cpu_count() or 1)


def _gpu(x, d, u, lam, z0, p2, m, incident="plane", x0=0.0, tol=1e-5):
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    xt = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()
    dt = torch.from_numpy(np.ascontiguousarray(d, dtype=np.float64)).cuda()
    plan = asf.LinePlan(xt, dt, lam, z0, p2, m, tol=tol, incident=incident, x0=x0)
    ut = torch.from_numpy(np.ascontiguousarray(u, dtype=np.complex64)).cuda()
    got = plan.forward(ut).cpu().numpy().astype(np.complex128)
    plan.close()
    return got


def _oracle(x, d, u, lam, z0, p2, m, incident="plane", x0=0.0):
    import oracle
    return oracle.line("eq7", x, d, np.asarray(u, dtype=np.complex64), lam, z0, p2, m,
                       incident=incident, nthreads=ORACLE_THREADS, x0=x0)


@pytest.mark.parametrize("name", synth.LINE_CONFIG_NAMES)
def test_paper_profiles(name):
    w = synth.line_config(name)
    got = _gpu(w.x, w.d, w.u, w.lam, w.z0, w.p2, w.m)
    err = rel_l2(got, _oracle(w.x, w.d, w.u, w.lam, w.z0, w.p2, w.m))
    print(f"{name}: n={w.n} m={w.m} rel-L2 {err:.3e}")
    assert err <= TOL


def _random_case(n, m, seed, spread=2e-3, lam=633e-9, z0=0.2):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-spread, spread, n)                       # unsorted, ragged n
    d = 40e-6 * np.sin(2 * np.pi * x / 0.9e-3) + rng.uniform(-5e-6, 5e-6, n)
    u = (rng.uniform(0, 1, n) * np.exp(2j * np.pi * rng.uniform(0, 1, n))).astype(np.complex64)
    return x, d, u, lam, z0


@pytest.mark.parametrize("incident,x0", [("plane", 0.0), ("none", 0.0), ("plane", 0.173e-3)])
def test_ragged_unsorted(incident, x0):
    x, d, u, lam, z0 = _random_case(1000, 64, 1)
    got = _gpu(x, d, u, lam, z0, 8e-6, 64, incident, x0)
    err = rel_l2(got, _oracle(x, d, u, lam, z0, 8e-6, 64, incident, x0))
    print(f"ragged {incident} x0={x0}: rel-L2 {err:.3e}")
    assert err <= TOL


def test_wrapping_frequencies():
    # p2 x / (lambda r0) spans several periods: the footprints wrap around the fine line
    x, d, u, lam, z0 = _random_case(700, 32, 2, spread=4e-2)
    got = _gpu(x, d, u, lam, z0, 8e-6, 32)
    err = rel_l2(got, _oracle(x, d, u, lam, z0, 8e-6, 32))
    print(f"wrapping: rel-L2 {err:.3e}")
    assert err <= TOL


def test_single_point_and_clustered():
    got = _gpu(np.array([37e-6]), np.array([3e-6]), np.array([0.6 - 0.3j]), 633e-9, 0.2, 8e-6, 16)
    want = _oracle(np.array([37e-6]), np.array([3e-6]), np.array([0.6 - 0.3j]), 633e-9, 0.2, 8e-6, 16)
    assert rel_l2(got, want) <= TOL
    # 3000 points inside one fine cell's width: every footprint overlaps every other
    rng = np.random.default_rng(3)
    x = rng.uniform(-2e-7, 2e-7, 3000)
    d = rng.uniform(0, 1e-6, 3000)
    u = (rng.standard_normal(3000) + 1j * rng.standard_normal(3000)).astype(np.complex64)
    got = _gpu(x, d, u, 633e-9, 0.2, 8e-6, 128)
    err = rel_l2(got, _oracle(x, d, u, 633e-9, 0.2, 8e-6, 128))
    print(f"clustered: rel-L2 {err:.3e}")
    assert err <= TOL


def test_largest_sizes():
    import paper_1203_3583_amd as asf

    n, m = asf.asf.LINE_MAX_POINTS, 8192
    x, d, u, lam, z0 = _random_case(n, m, 4, spread=6e-3, z0=0.5)
    p2 = 4e-6
    got = _gpu(x, d, u, lam, z0, p2, m)
    ix = np.concatenate([np.arange(0, 64), np.arange(m // 2 - 64, m // 2 + 64), np.arange(m - 64, m),
                         np.random.default_rng(5).choice(m, 256, replace=False)])
    import oracle
    want = oracle.line("eq7", x, d, u, lam, z0, p2, m, ix=ix, nthreads=ORACLE_THREADS)
    err = rel_l2(got[ix], want)
    print(f"n={n} m={m}: rel-L2 {err:.3e} on {len(ix)} pixels")
    assert err <= TOL


def test_accuracy_follows_tolerance():
    x, d, u, lam, z0 = _random_case(900, 128, 6)
    want = _oracle(x, d, u, lam, z0, 8e-6, 128)
    for tol in (1e-3, 1e-4, 1e-6):
        err = rel_l2(_gpu(x, d, u, lam, z0, 8e-6, 128, tol=tol), want)
        print(f"tol {tol:g}: rel-L2 {err:.3e}")
        assert err <= max(tol, 2e-6)


def test_batch_matches_single_calls_bitwise():
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    x, d, _, lam, z0 = _random_case(500, 256, 7)
    rng = np.random.default_rng(8)
    us = (rng.standard_normal((3, 500)) + 1j * rng.standard_normal((3, 500))).astype(np.complex64)
    plan = asf.LinePlan(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), lam, z0, 8e-6, 256)
    ub = torch.from_numpy(us).cuda()
    batch = plan.forward(ub).cpu().numpy()
    again = plan.forward(ub).cpu().numpy()
    singles = np.stack([plan.forward(ub[b].contiguous()).cpu().numpy() for b in range(3)])
    plan.close()
    assert np.array_equal(batch.view(np.uint32), again.view(np.uint32))
    assert np.array_equal(batch.view(np.uint32), singles.view(np.uint32))
    for b in range(3):
        assert rel_l2(batch[b], _oracle(x, d, us[b], lam, z0, 8e-6, 256)) <= TOL


def test_domain_error_reported():
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    x = torch.zeros(4, dtype=torch.float64, device="cuda")
    d = torch.tensor([0.0, 0.0, 0.25, 0.0], dtype=torch.float64, device="cuda")
    with pytest.raises(asf.AsfError) as e:
        asf.LinePlan(x, d, 633e-9, 0.2, 8e-6, 16)
    assert e.value.code == asf.asf.ASF_EDOMAIN


@pytest.mark.parametrize("n,m,batch,spread", [
    (1, 16, 1, 2e-3),         # one point, fields of the workgroup missing
    (3000, 16, 9, 2e-7),      # every point in one cell, the fields too large for LDS, a ragged last workgroup
    (37, 32, 5, 4e-2),        # wrapping, fewer points than cells
    (5200, 64, 3, 2e-3),
    (700, 128, 1, 2e-7),
    (4099, 128, 600, 2e-3),
    (900, 256, 2049, 2e-3),   # two fields per workgroup, a ragged last one
    (11000, 512, 300, 2e-3),  # too large for LDS
    (6000, 512, 1, 2e-7),
    (333, 1024, 2049, 2e-3),  # the first length a thread per cell gathers
    (9000, 1024, 300, 2e-7),
])
def test_gather_paths(n, m, batch, spread):
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    x, d, _, lam, z0 = _random_case(n, 0, 11, spread=spread)
    rng = np.random.default_rng(12)
    us = (rng.standard_normal((batch, n)) + 1j * rng.standard_normal((batch, n))).astype(np.complex64)
    plan = asf.LinePlan(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), lam, z0, 8e-6, m, tol=1e-5)
    ub = torch.from_numpy(us).cuda()
    got = plan.forward(ub)
    again = plan.forward(ub)
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(again))
    got = got.cpu().numpy()
    plan.close()
    for b in sorted({0, batch // 2, batch - 1}):
        assert rel_l2(got[b], _oracle(x, d, us[b], lam, z0, 8e-6, m)) <= TOL


@pytest.mark.parametrize("n,m,batch", [
    (6000, 1024, 2049),   # a thread per cell
    (7000, 256, 2049),    # shared runs
    (5500, 512, 2050),
])
def test_two_fields_per_workgroup_too_large_for_lds(n, m, batch):
    """Batches of 2048 fields and more, two to a workgroup, gathered from memory: the first
    and the last fields (with an odd batch the last workgroup has one) and one in between
    against the oracle, and the same as each alone."""
    torch = torch_gpu()
    import paper_1203_3583_amd as asf

    x, d, _, lam, z0 = _random_case(n, 0, 21, spread=2e-3)
    plan = asf.LinePlan(torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), lam, z0, 8e-6, m, tol=1e-5)
    g = torch.Generator(device="cuda").manual_seed(22)
    ub = torch.view_as_complex(torch.randn((batch, n, 2), generator=g, device="cuda"))
    got = plan.forward(ub)
    for b in (0, 1, 1001, batch - 2, batch - 1):
        u = ub[b].contiguous()
        assert rel_l2(got[b].cpu().numpy(), _oracle(x, d, u.cpu().numpy(), lam, z0, 8e-6, m)) <= TOL
        assert rel_l2(got[b].cpu().numpy(), plan.forward(u).cpu().numpy()) <= TOL
    plan.close()
