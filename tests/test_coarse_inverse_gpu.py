"""The coarsest level's inverse, formed on the device.

A hierarchy with one level solves A x = b with the inverse alone, so one cycle
from zero gives the inverse applied to b.  The sizes cover the one-workgroup
form (n <= 192) at the edges of its 32-row tiles and the blocked form above,
with ragged last blocks, every boundary rule and both coefficient modes, and a
two-level case in which a coefficient update goes through the blocked form.
The bar is the error of a backward-stable solve in double precision: the
condition number of these matrices is below 1e3, and n times that times eps
below 1e-10.
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N, P = 0, 1, 2
BCS = {"dirichlet": (D,) * 6, "neumann": (N,) * 6, "top": (N, N, N, N, N, D), "mixed": (P, P, D, N, N, N)}


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


def coefficient(shape, seed):
    return 10.0 ** np.random.default_rng(seed).uniform(-1.5, 1.5, size=shape[::-1])


def check(H, OH, b, tol):
    x = dev(np.zeros_like(b))
    info = H.solve(dev(b), x, max_cycles=1, fixed_cycles=True)
    xo, _, st = OH.solve(b, max_cycles=1, fixed=True)
    assert st == 0 and info.cycles == 1
    err = np.max(np.abs(x.cpu().numpy().reshape(b.shape) - xo)) / np.max(np.abs(xo))
    assert err <= tol, err


@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 1, 5), (4, 4, 2), (3, 11, 1), (4, 4, 4), (5, 13, 1), (5, 5, 5),
                                   (4, 8, 6), (13, 3, 5), (5, 6, 7), (4, 6, 10), (7, 8, 8), (8, 8, 8)])
@pytest.mark.parametrize("nodal", [False, True])
def test_one_level_solve_is_the_inverse(mg, shape, bc, nodal):
    k = coefficient(shape, 3) if nodal else None
    b = inputs.gaussian(shape, 5, zero_mean=False)
    h = 0.25
    cfg = mg.config_default(*shape, h, bc=BCS[bc], coef_mode=1 if nodal else 0, min_coarse=512)
    if shape == (1, 1, 1) and D not in BCS[bc]:  # the operator is zero: no inverse
        with pytest.raises(mg.Nn4mgError):
            mg.Hierarchy(cfg, dev(k) if nodal else None)
        return
    H = mg.Hierarchy(cfg, dev(k) if nodal else None)
    assert len(H.levels()) == 1
    OH = oracle.Hierarchy(shape, h, BCS[bc], k=k, min_coarse=512)
    check(H, OH, b, 1e-10)


@pytest.mark.parametrize("precision", [0, 1])
def test_update_through_the_blocked_inverse(mg, precision):
    shape, bc, h = (16, 24, 40), BCS["top"], 1.0 / 16
    k1, k2 = coefficient(shape, 7), coefficient(shape, 8)
    b = inputs.gaussian(shape, 9, zero_mean=False)
    cfg = mg.config_default(*shape, h, bc=bc, coef_mode=1, precision=precision)
    H = mg.Hierarchy(cfg, dev(k1))
    assert H.levels()[-1] == (4, 6, 10)
    H.update_coef(dev(k2))
    check(H, oracle.Hierarchy(shape, h, bc, k=k2), b, 1e-10 if precision == 0 else 1e-5)
    bad = k2.copy()
    bad[3, 4, 5] = -1.0
    with pytest.raises(mg.Nn4mgError):
        H.update_coef(dev(bad))
    H.update_coef(dev(k1))
    check(H, oracle.Hierarchy(shape, h, bc, k=k1), b, 1e-10 if precision == 0 else 1e-5)
