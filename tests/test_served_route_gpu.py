"""Which coarse end a server's requests run: with the coarse end's matrix where a
full group that way takes at most an eighth of the budget, or where the matrix is
at most a 32nd of the copy's other bytes and the budget holds a full group; below,
without it, so the matrices do not take the room of copies.  Told by the memory at
its peak, which is the group's: as many copies as requests may run, each with its
right-hand side and iterate and at most the bytes that are reported for its
hierarchy (kilobytes less, for alignment).  The results are the same to the
solve's tolerance.
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("edge,cells,share", [(32, 512, 8), (96, 216, 1)])  # cells of the matrix's level
@pytest.mark.parametrize("slots", [1, 3])
def test_matrix_follows_the_budget(edge, cells, share, slots):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    shape, bc = (edge,) * 3, (1,) * 6
    h, n = 1.0 / edge, edge ** 3
    frac = inputs.sphere_fraction(shape, h, [0.5] * 3, 0.3)
    k = inputs.two_phase_k(frac, 100.0, 1.0)
    b = inputs.gaussian(shape, 5, zero_mean=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).cuda()
    cfg = mg.config_default(*shape, h, bc=bc, coef_mode=1, precision=1)
    matrix = 8 * cells * cells
    full = mg.bytes_required(cfg) + 16 * n
    assert (32 * matrix <= full - matrix) == (share == 1)
    kd, bd = dev(k), dev(b)
    for budget, taken in [(share * slots * full, True), (share * slots * full - 1, False)]:
        srv = mg.Server(budget, slots)
        xs = [dev(np.zeros_like(b)) for _ in range(2 * slots)]
        for i, x in enumerate(xs):
            srv.submit(cfg, bd, x, k=kd, rtol=1e-8, max_cycles=500, tag=i)
        srv.drain()
        assert all(r.info.status == 0 for r in srv.poll())
        peak, low = srv.stats()["peak_bytes"], slots * (full - matrix)
        assert (low < peak <= slots * full) if taken else (0.9 * low < peak <= low)
        srv.close()
        for x in xs:
            r = b - oracle.apply(x.cpu().numpy().reshape(b.shape), h, bc, k)
            assert np.linalg.norm(r) <= 1.05e-8 * np.linalg.norm(b)
