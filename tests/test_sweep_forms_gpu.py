"""The two forms of the two-sweep pass (a march over z, independent blocks) give
the same bits: both go through the same operations in the same order, so a
level may take either, per launch, without changing a result.

One cycle with the marching form on every level, and with blocks on every level,
the finest included (in FP64 from x + P e with the projected right-hand side),
over ragged grids, every boundary rule, precision and coefficient mode; the FP64
cycle also against the oracle's to the single-cycle bar of 1e-12.
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N, P = 0, 1, 2


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


@pytest.mark.parametrize("shape", [(8, 8, 8), (40, 12, 24), (20, 28, 36), (64, 64, 64), (96, 80, 48)])
@pytest.mark.parametrize("bc", [(N,) * 6, (D, N, P, P, N, D)])
@pytest.mark.parametrize("precision,nodal", [(0, False), (0, True), (1, False), (1, True), (2, True)])
def test_march_and_blocks_agree_bitwise(mg, shape, bc, precision, nodal):
    h = 1.0 / shape[0]
    k = 10.0 ** np.random.default_rng(4).uniform(-1.5, 1.5, size=shape[::-1]) if nodal else None
    b, x0 = inputs.gaussian(shape, 5, zero_mean=True), inputs.gaussian(shape, 6, zero_mean=False)
    cfg = mg.config_default(*shape, h, bc=bc, coef_mode=1 if nodal else 0, precision=precision)
    H = mg.Hierarchy(cfg, dev(k) if nodal else None)
    out = []
    for tile in ((32, 2, 4), (16, 2, 2), (8, 8, 8)):
        for l, d in enumerate(H.levels()[:-1]):
            if min(d) >= 4:
                H.set_tiles(l, *tile, kclass=mg.KCLASS_FINE_SWEEP_PROLONG)
        x = dev(x0)
        H.vcycle(dev(b), x)
        y = dev(np.zeros_like(b))  # a solve: with the mean of b taken off where the problem is singular
        H.solve(dev(b + 0.25), y, max_cycles=3, fixed_cycles=True)
        out.append((x.cpu().numpy(), y.cpu().numpy()))
    for x, y in out[1:]:
        assert np.array_equal(x, out[0][0]) and np.array_equal(y, out[0][1])
    if precision == 0:
        want = oracle.Hierarchy(shape, h, bc, k=k).vcycle(x0, b)
        assert np.max(np.abs(out[0][0].reshape(b.shape) - want)) <= 1e-12 * np.max(np.abs(want))
