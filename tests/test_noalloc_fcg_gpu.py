"""The allocation-free residual of a flexible-CG configuration around an FP32
cycle, whose hierarchy gives its residual another launch shape than the default
rule: the contract is the same kernel in the same shape, so r and the norm are
the hierarchy's bit for bit.  Grids where the two shapes differ (other chunks of
planes, other tile widths), with the other precisions and the stationary
iteration beside them.
"""
import numpy as np
import pytest

from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N = 0, 1


@pytest.mark.parametrize("shape", [(128, 96, 96), (96, 64, 160), (80, 48, 112), (24, 16, 40)])
@pytest.mark.parametrize("outer,precision", [(1, 0), (1, 1), (1, 2), (0, 1)])
def test_same_residual_and_norm(shape, outer, precision):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    h = 1.0 / shape[0]
    cfg = mg.config_default(*shape, h, bc=(N, N, N, N, N, D), coef_mode=1, precision=precision, outer=outer)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).cuda()
    k = dev(np.exp(np.random.default_rng(1).uniform(-2.0, 2.0, size=shape[::-1])))
    H = mg.Hierarchy(cfg, k)
    for seed in range(4):
        x, b = (dev(inputs.gaussian(shape, 2 * seed + q, zero_mean=False)) for q in (0, 1))
        r0, r1 = torch.empty_like(x), torch.empty_like(x)
        n0 = H.residual(x, b, r0)
        n1 = mg.residual_noalloc(cfg, x, b, k=k, r=r1)
        assert torch.equal(r0, r1)
        assert n0 == n1, (seed, n0, n1)
