"""The flexible-CG iterate x when an iteration's update is deferred to its end.

However the solve ends (the tolerance inside a batch of iterations, the
iteration limit, a fixed count), x must hold every update: the oracle's residual
of x equals the recurrence's last residual.  For the one-pass sweeps (z in FP32
with a mixed cycle) and for one sweep per pass (z in FP64).  The recurrence's
residual drifts from the true one by rounding only: 1e-12 of ||b||.
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N = 0, 1


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


@pytest.mark.parametrize("shape,bc", [((16, 16, 16), (N, N, N, N, N, D)), ((40, 24, 32), (D,) * 6),
                                      ((64, 64, 64), (N,) * 6)])
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("nu", [1, 2])
def test_iterate_holds_every_update(mg, shape, bc, precision, nu):
    h = 1.0 / shape[0]
    frac = inputs.sphere_fraction(shape, h, [0.5 * n * h for n in shape], 0.3 * min(shape) * h)
    k = inputs.two_phase_k(frac, 1000.0, 1.0)
    b = inputs.gaussian(shape, 11, zero_mean=True)
    cfg = mg.config_default(*shape, h, bc=bc, coef_mode=1, precision=precision, outer=mg.OUTER_FCG, nu_post=nu)
    H = mg.Hierarchy(cfg, dev(k))
    for kw in (dict(rtol=1e-6, max_cycles=60), dict(rtol=1e-12, max_cycles=3), dict(rtol=0.0, max_cycles=5, fixed_cycles=True)):
        x = dev(np.zeros_like(b))
        info = H.solve(dev(b), x, **kw)
        r = b - oracle.apply(x.cpu().numpy().reshape(b.shape), h, bc, k)
        assert abs(np.linalg.norm(r) / np.linalg.norm(b) - info.relres) <= 1e-12 + 1e-9 * info.relres, (kw, info.cycles)
