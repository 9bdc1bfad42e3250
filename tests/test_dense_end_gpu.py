"""The coarse end of the cycle as one matrix (its levels' restriction, exact
solve, prolongation and sweeps composed when the coefficient is set).

One cycle and a solve of five cycles (whose stopping rule runs in the product's
launch when no restriction chain precedes it) against the oracle, at the edges
of the product's tiles (16 rows, 512 and 1024 columns), with the matrix on the
first, second, third and fourth level below the finest, in every precision, for
a stand-alone hierarchy and through the server (copies of one group).
Bars: those of the repository's single cycle (1e-12 of the largest entry in
FP64; 2e-5 of the largest correction with FP32 smoothing, 2e-2 with FP16
coefficients) and of its fixed-count solves (1e-10).
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N, P = 0, 1, 2
BCS = {"dirichlet": (D,) * 6, "neumann": (N,) * 6, "mixed": (N, D, P, P, N, N)}
SHAPES = [(8, 8, 8), (6, 10, 14), (16, 16, 16), (20, 20, 20), (16, 32, 16), (24, 40, 32), (64, 64, 64), (128, 64, 64)]


@pytest.fixture(scope="module")
def mg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg

    nn4mg.lib()
    return nn4mg


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64).reshape(-1)).cuda()


def work(shape, nodal):
    h = 1.0 / shape[0]
    k = None
    if nodal:
        frac = inputs.sphere_fraction(shape, h, [0.5 * n * h for n in shape], 0.3 * min(shape) * h)
        k = inputs.two_phase_k(frac, 100.0, 1.0)
    return h, k, inputs.gaussian(shape, 5, zero_mean=True), inputs.gaussian(shape, 6, zero_mean=True)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("nodal", [False, True])
def test_cycle_and_solve_fp64(mg, shape, bc, nodal):
    h, k, b, x0 = work(shape, nodal)
    cfg = mg.config_default(*shape, h, bc=BCS[bc], coef_mode=1 if nodal else 0)
    H = mg.Hierarchy(cfg, dev(k) if nodal else None)
    OH = oracle.Hierarchy(shape, h, BCS[bc], k=k)
    x = dev(x0)
    H.vcycle(dev(b), x)
    want = OH.vcycle(x0.copy(), b)
    assert np.max(np.abs(x.cpu().numpy().reshape(b.shape) - want)) <= 1e-12 * np.max(np.abs(want))
    x = dev(np.zeros_like(b))
    info = H.solve(dev(b), x, max_cycles=5, fixed_cycles=True)
    xo, hist, st = OH.solve(b, max_cycles=5, fixed=True)
    assert st == 0 and info.cycles == 5
    np.testing.assert_allclose(info.history(), hist, rtol=1e-10, atol=1e-13)
    assert np.max(np.abs(x.cpu().numpy().reshape(b.shape) - xo)) <= 1e-10 * np.max(np.abs(xo))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("precision,nodal,tol", [(1, False, 2e-5), (1, True, 2e-5), (2, True, 2e-2)])
def test_cycle_mixed(mg, shape, precision, nodal, tol):
    h, k, b, x0 = work(shape, nodal)
    cfg = mg.config_default(*shape, h, bc=BCS["mixed"], coef_mode=1 if nodal else 0, precision=precision)
    H = mg.Hierarchy(cfg, dev(k) if nodal else None)
    x = dev(x0)
    H.vcycle(dev(b), x)
    want = oracle.Hierarchy(shape, h, BCS["mixed"], k=k).vcycle(x0.copy(), b)
    assert np.max(np.abs(x.cpu().numpy().reshape(b.shape) - want)) <= tol * np.max(np.abs(want - x0))


@pytest.mark.parametrize("budget", [8 << 30, 6 << 20])
def test_served_with_and_without_the_matrix(mg, budget):
    """A budget too small for a group with matrices serves without them."""
    shape, bc = (32, 32, 32), BCS["neumann"]
    h, k, b, _ = work(shape, True)
    cfg = mg.config_default(*shape, h, bc=bc, coef_mode=1, precision=1)
    srv = mg.Server(budget, 3)
    xs = [dev(np.zeros_like(b)) for _ in range(3)]
    kd, bd = dev(k), dev(b)
    for i, x in enumerate(xs):
        srv.submit(cfg, bd, x, k=kd, rtol=1e-8, max_cycles=500, tag=i)
    srv.drain()
    assert all(r.info.status == 0 for r in srv.poll())
    assert srv.stats()["peak_bytes"] <= budget
    srv.close()
    for x in xs:
        r = b - oracle.apply(x.cpu().numpy().reshape(b.shape), h, bc, k)
        assert np.linalg.norm(r) <= 1.05e-8 * np.linalg.norm(b)
