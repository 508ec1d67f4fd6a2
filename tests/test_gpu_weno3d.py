"""3D stages with every face WENO (one kernel per direction) against the stage
kernel with per-cell corrections."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say, to_dev, to_host
from paper_1908_02464_amd import workloads as w

pytestmark = pytest.mark.gpu


def _noisy(nx, ny, nz):
    """A smooth flow with pressure and density jumps and noise."""
    r = np.random.default_rng(nx * 10000 + ny * 100 + nz)
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    jump = ((x + 2 * y + 3 * z) // 5) % 3
    rho = 1.0 + 0.5 * jump + 0.1 * r.random(x.shape)
    vel = [0.3 * np.sin(0.7 * c + k) + 0.2 * r.standard_normal(x.shape) for k, c in enumerate((x, y, z))]
    p = 1.0 + jump + 0.1 * r.random(x.shape)
    return w.conserved(rho, vel, p), 1.0 / max(nx, ny, nz)


# rows of faces against 63 per wavefront, columns against 64, chunks against the
# grid (march 0: chosen, 1, one that leaves a remainder, one beyond the grid)
@pytest.mark.parametrize("split", [0, 1, 2])
@pytest.mark.parametrize("shape,bc,weights,march", [
    ((2, 3, 2), [0, 0, 2, 2, 1, 1], 0, 0), ((5, 2, 4), [1, 1, 0, 0, 0, 0], 0, 1),
    ((62, 5, 7), [0, 0, 2, 2, 1, 1], 0, 3), ((63, 4, 6), [2, 1, 1, 2, 0, 0], 1, 0),
    ((64, 7, 3), [1, 2, 0, 0, 1, 2], 2, 2), ((65, 33, 17), [0, 0, 0, 0, 0, 0], 0, 0),
    ((130, 9, 20), [2, 2, 1, 1, 2, 1], 0, 7), ((31, 40, 70), [0, 0, 1, 2, 0, 0], 2, 100)])
def test_weno3d_bitwise(shape, bc, weights, march, split):
    import torch
    from paper_1908_02464_amd import capi
    nx, ny, nz = shape
    U, dx = _noisy(nx, ny, nz)
    say(f"[weno3d] {shape} bc={bc} weights={weights} march={march} split={split}")
    res = []
    for path, chunk in ((0, march), (3, 0)):  # 3: per-cell corrections
        p = capi.params_default(nx, ny, nz, dx, bc=bc, hybrid=2, weights=weights, split=split)
        ctx = capi.Context(nx, ny, nz, dx, 1.4, p)
        ctx.tune(path, chunk)
        A = to_dev(U)
        D = torch.full_like(A, float("nan"))
        ctx.rhs(A, D)
        ctx.step(A)
        ctx.advance(A, 3, 1e300)
        torch.cuda.synchronize()
        assert ctx.status() == 0
        res.append((to_host(D), to_host(A), ctx.clock()))
        ctx.close()
    assert np.array_equal(res[0][0], res[1][0])
    assert np.array_equal(res[0][1], res[1][1])
    assert res[0][2] == res[1][2]
