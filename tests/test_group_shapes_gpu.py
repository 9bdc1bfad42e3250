"""A batched group's two-sweep passes take their launch shapes from the number of
copies that a launch covers, the residual from a fixed one, so a request's result
does not depend on who runs beside it, and a request alone is not slowed down by
shapes meant for several.

Bits: the same requests one at a time, in groups of at most three copies and all
at once, over grids where one, two and four copies get different forms (blocks or
march), tile widths and chunks.  Time: a 96^3 request alone in a group against
the same update and solve on a hierarchy of its own.  The group's cycle moves a
third more bytes in FP64 (the full residual) and adds the admission's copies;
measured 1.24 (FP64) and 1.27 (FP32 smoothing), with shapes for four copies 1.59
and 1.65, so the bar is 1.42, half way.
"""
import time

import numpy as np
import pytest

from paper_2401_06755_amd import inputs

pytestmark = pytest.mark.gpu

N, D = 1, 0


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

    return torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).cuda()


@pytest.mark.parametrize("shape", [(48, 48, 48), (40, 64, 48), (80, 48, 112), (96, 96, 96)])
@pytest.mark.parametrize("precision,nodal", [(0, True), (0, False), (1, True), (2, True)])
def test_same_bits_whoever_runs_beside(mg, shape, precision, nodal):
    import torch

    h = 1.0 / shape[0]
    cfg = mg.config_default(*shape, h, bc=(N, N, N, N, N, D), coef_mode=1 if nodal else 0, precision=precision)
    ks = [dev(np.exp(np.random.default_rng(s).uniform(-1, 1, size=shape[::-1]))) if nodal else None for s in range(6)]
    bs = [dev(inputs.gaussian(shape, 20 + s, zero_mean=False)) for s in range(6)]
    out = []
    for slots in (1, 3, 6):
        srv = mg.Server(16 << 30, slots)
        xs = [torch.zeros_like(b) for b in bs]
        for i, x in enumerate(xs):
            srv.submit(cfg, bs[i], x, k=ks[i], rtol=1e-7, max_cycles=400, tag=i)
        srv.drain()
        assert all(r.info.status == 0 for r in srv.poll())
        srv.close()
        out.append(xs)
    for xs in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(xs, out[0]))


@pytest.mark.parametrize("precision", [0, 1])
def test_request_alone_in_a_group(mg, precision):
    import torch

    shape, h = (96, 96, 96), 1.0 / 96
    frac = inputs.sphere_fraction(shape, h, [0.5] * 3, 0.3)
    k, b = dev(inputs.two_phase_k(frac, 100.0, 1.0)), dev(inputs.gaussian(shape, 5, zero_mean=True))
    cfg = mg.config_default(*shape, h, bc=(N,) * 6, coef_mode=1, precision=precision)
    H, srv = mg.Hierarchy(cfg, k), mg.Server(16 << 30, 8)
    own, served = 1e9, 1e9
    for _ in range(8):
        x, y = torch.zeros_like(b), torch.zeros_like(b)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        H.update_coef(k)
        H.solve(b, x, rtol=1e-8, max_cycles=500)
        torch.cuda.synchronize()
        own = min(own, 1e3 * (time.perf_counter() - t0))
        srv.submit(cfg, b, y, k=k, rtol=1e-8, max_cycles=500)
        srv.drain()
        r = srv.poll()[0]
        served = min(served, r.t_done_ms - r.t_start_ms)
    srv.close()
    assert served <= 1.42 * own, (served, own)
