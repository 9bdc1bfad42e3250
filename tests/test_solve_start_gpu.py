"""The first residual of a solve, judged in the first cycle's own launches.

A start that already meets the tolerance leaves x as it was (no cycle counted;
bit for bit, or for a singular problem, which ends with the mean taken off, but
for that constant and its rounding, half an ulp of |x| < 8), a zero right-hand side ends at once, a limit of one cycle stops
after one, and a new solve on the same handle begins with a cleared state.  With
and without a coarse chain (two and five levels), singular and not, against the
oracle's first residual (1e-12 relative: sums of the same terms in another order).
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N = 0, 1


@pytest.mark.parametrize("shape", [(8, 6, 10), (48, 32, 64)])
@pytest.mark.parametrize("bc", [(D,) * 6, (N,) * 6])
@pytest.mark.parametrize("precision", [0, 1])
def test_first_residual(shape, bc, precision):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    h = 1.0 / shape[0]
    b = inputs.gaussian(shape, 3, zero_mean=True)
    x0 = inputs.gaussian(shape, 4, zero_mean=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64).reshape(-1)).cuda()
    H = mg.Hierarchy(mg.config_default(*shape, h, bc=bc, precision=precision))
    bd, x = dev(b), dev(x0)
    first = np.linalg.norm(b - oracle.apply(x0, h, bc, None)) / np.linalg.norm(b)
    for _ in range(2):  # the second solve starts from a cleared state
        x = dev(x0)
        info = H.solve(bd, x, rtol=2.0 * first)
        assert info.cycles == 0 and info.status == 0
        off = x - dev(x0)
        assert float(off.max() - off.min()) <= (1e-15 if bc[0] == N else 0.0)
        assert abs(info.relres - first) <= 1e-12 * first
        info = H.solve(bd, x, rtol=1e-30, max_cycles=1)
        assert info.cycles == 1 and len(info.history()) == 2
        assert abs(info.history()[0] - first) <= 1e-12 * first and info.relres < first
    zero = torch.zeros_like(bd)
    x = zero.clone()
    info = H.solve(zero, x)
    assert info.cycles == 0 and info.relres == 0.0 and torch.equal(x, zero)
