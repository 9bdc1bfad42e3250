"""The linear step with several output planes per workgroup: a flow in motion on
grids ragged in x and y whose z-march runs in chunks that do not divide nz, so
the running sums are carried from plane to plane, the two LDS buffers are used
over and over and the last chunk is shorter.  One step against the oracle, every
field; the bar is the step's own, 1e-9 of each field's largest value.

The chunk follows from a rule on the grid (fewest rounds of 512 workgroups times
steps), repeated here to see that the shapes are what this test is for.
"""
import numpy as np
import pytest

import oracle
from tests.test_step_march_gpu import moving_state

pytestmark = pytest.mark.gpu


def chunk(shape, rows):
    nx, ny, nz = shape
    tiles = -(-nx // 32) * -(-ny // (8 * rows))
    best, zc = float("inf"), 1
    for c in range(1, min(nz, 128) + 1):
        rounds, rest = divmod(tiles * -(-nz // c), 512)
        cost = (rounds + (0.0 if rest == 0 else 0.7 if rest <= 256 else 1.0)) * (c + 2)
        if cost < best:
            best, zc = cost, c
    return zc


@pytest.mark.parametrize("shape,chunks", [((40, 40, 104), (5, 3)), ((72, 56, 56), (5, 3)), ((112, 80, 112), (10, 5))])
def test_one_step_over_chunks(shape, chunks):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg as mg

    assert (chunk(shape, 1), chunk(shape, 2)) == chunks
    assert all(c >= 3 and shape[2] % c for c in chunks)
    h, st = moving_state(*shape)
    kw = dict(rho_g=500.0, dt=1e-4, mg_cycles=12, n_corr=2, n_vel_iter=2)
    dev = {k: torch.from_numpy(a.reshape(-1).copy()).cuda() for k, a in st.items()}
    info = mg.Stepper(*shape, h, mg.step_params(**kw)).step(dev)
    oracle.step(st, h, oracle.step_params(**kw))
    for k, a in st.items():
        got = dev[k].cpu().numpy().reshape(a.shape)
        assert np.max(np.abs(got - a)) <= 1e-9 * np.max(np.abs(a)), k
    assert abs(info.volume - st["C"].sum() * h ** 3) <= 1e-10 * abs(info.volume)
