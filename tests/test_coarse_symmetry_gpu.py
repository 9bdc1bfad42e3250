"""The coarsest inverse is stored exactly symmetric: the cycle reads its columns
as rows, and flexible CG expects a symmetric preconditioner.  A hierarchy with
one level applies the inverse alone, so a cycle from zero on a unit vector gives
a column of it, entry by entry (every other product is an exact zero).  Sizes of
the one-workgroup form (n <= 192) and of the blocked one, with ragged tiles.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

D, N, P = 0, 1, 2


@pytest.mark.parametrize("shape", [(3, 2, 2), (5, 5, 5), (4, 6, 8), (5, 6, 7), (7, 8, 6)])
@pytest.mark.parametrize("bc", [(D,) * 6, (P, P, N, N, N, D)])
def test_inverse_is_symmetric(shape, bc):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    n = int(np.prod(shape))
    k = 10.0 ** np.random.default_rng(4).uniform(-1.5, 1.5, size=n)
    cfg = mg.config_default(*shape, 0.25, bc=bc, coef_mode=1, min_coarse=512)
    H = mg.Hierarchy(cfg, torch.from_numpy(k).cuda())
    assert len(H.levels()) == 1
    unit = torch.eye(n, dtype=torch.float64, device="cuda")
    inv = torch.zeros_like(unit)
    for j in range(n):
        H.vcycle(unit[j], inv[j])
    assert torch.equal(inv, inv.T.contiguous()), float((inv - inv.T).abs().max())
