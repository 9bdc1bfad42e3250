"""The linear step at the edges of the z-march's tiles (32 cells along x, 8 or 16
along y, chunks of planes): grids smaller than a tile, ragged in every direction
and with more than one chunk, one step against the oracle with the velocity and
pressures of a flow in motion.  The bar is the step's own: 1e-9 of each field's
largest value.
"""
import numpy as np
import pytest

import oracle
from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2401_06755_amd import nn4mg

    nn4mg.lib()
    return nn4mg


def moving_state(nx, ny, nz):
    h = 1.0 / nx
    C = 1.0 - inputs.sphere_fraction((nx, ny, nz), h, (0.45, 0.5 * ny * h, 0.4 * nz * h), 0.3 * min(nx, ny, nz) * h)
    x, y, z = (np.pi * (np.arange(n) + 0.5) / n for n in (nx, ny, nz))
    def outer(fz, fy, fx):
        return fz(z / 2)[:, None, None] * fy(y)[None, :, None] * fx(x)[None, None, :]

    u, v, w = 0.3 * outer(np.cos, np.cos, np.sin), -0.1 * outer(np.cos, np.sin, np.cos), 0.2 * outer(np.sin, np.cos, np.cos)
    p = 9810.0 * h * (nz - np.arange(nz) - 0.5)[:, None, None] * np.ones((nz, ny, nx))
    pn = 5.0 * inputs.gaussian((nx, ny, nz), 3, zero_mean=False)
    return h, {k: np.ascontiguousarray(a) for k, a in dict(C=C, u=u, v=v, w=w, p_hs=p, p_nh=pn).items()}


@pytest.mark.parametrize("shape", [(4, 4, 4), (8, 4, 12), (12, 20, 28), (40, 24, 16), (72, 40, 24), (32, 16, 64)])
@pytest.mark.parametrize("order", [1, 2])
def test_one_step_on_ragged_grids(mg, shape, order):
    import torch

    h, st = moving_state(*shape)
    kw = dict(rho_g=500.0, dt=1e-4, mg_cycles=12, n_corr=2, n_vel_iter=2, order=order)
    dev = {k: torch.from_numpy(a.reshape(-1).copy()).cuda() for k, a in st.items()}
    info = mg.Stepper(*shape, h, mg.step_params(**kw)).step(dev)
    oracle.step(st, h, oracle.step_params(**kw))
    for k, a in st.items():
        got = dev[k].cpu().numpy().reshape(a.shape)
        assert np.max(np.abs(got - a)) <= 1e-9 * np.max(np.abs(a)), k
    assert abs(info.volume - st["C"].sum() * h ** 3) <= 1e-10 * abs(info.volume)
