"""Flexible CG around an FP32 cycle keeps the one-workgroup coarse end and its own
residual shape (64-wide tiles from 64 cells on, a power-of-two chunk of at most
64 planes that keeps 512 workgroups); the other configurations of the same grid
take the dense coarse end and the marching rule.

Checked by the memory each asks for (the matrix of the coarse end), by the shape
reported, and by five iterations on ragged grids against the oracle's residual
of the iterate (1e-12 of ||b||: the recurrence drifts by FP64 rounding only).
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

D, N = 0, 1


@pytest.mark.parametrize("shape,tile", [((48, 40, 32), None), ((64, 24, 40), (64, 2, 2)), ((128, 96, 96), (64, 2, 4))])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_route_and_iterate(shape, tile, precision):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    h, n = 1.0 / shape[0], int(np.prod(shape))
    bc = (N, N, N, N, N, D)

    def config(outer):
        return mg.config_default(*shape, h, bc=bc, coef_mode=1, precision=precision, outer=outer)

    # beyond the matrix, flexible CG holds four vectors and two rows of 1024 partial sums
    matrix = mg.bytes_required(config(mg.OUTER_STATIONARY)) - (mg.bytes_required(config(mg.OUTER_FCG)) - 32 * n - 16384)
    levels = [n >> (3 * l) for l in range(1, 8)]
    assert matrix in ([0] if precision == 0 else [8 * c * c for c in levels if c <= 1024])

    frac = inputs.sphere_fraction(shape, h, [0.5 * m * h for m in shape], 0.3 * min(shape) * h)
    k = inputs.two_phase_k(frac, 100.0, 1.0)
    b = inputs.gaussian(shape, 21)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64).reshape(-1)).cuda()
    H = mg.Hierarchy(config(mg.OUTER_FCG), dev(k))
    if precision and tile:
        t = H.get_tiles(0, mg.KCLASS_FINE_RESID)
        assert tuple(t) == tile
    x = dev(np.zeros_like(b))
    info = H.solve(dev(b), x, rtol=0.0, max_cycles=5, fixed_cycles=True)
    r = b - oracle.apply(x.cpu().numpy().reshape(b.shape), h, bc, k)
    assert abs(np.linalg.norm(r) / np.linalg.norm(b) - info.relres) <= 1e-12 + 1e-9 * info.relres
