"""2D row kernel: correction lists longer than a wavefront's buffer, and any
number of rows per item."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say, to_dev, to_host
from paper_1908_02464_amd import workloads as w

pytestmark = pytest.mark.gpu


# every cell flagged (noise): 63 entries per row of an item against a buffer of
# 256 that is emptied beyond 192; edges of the 63-column tiles
@pytest.mark.parametrize("nx,ny", [(62, 40), (63, 67), (127, 90), (400, 131)])
@pytest.mark.parametrize("kw", [{}, {"split": 1}, {"hybrid": 1}])
def test_rows_per_item_bitwise(nx, ny, kw):
    import torch
    from paper_1908_02464_amd import capi
    U, dx, _ = w.four_quadrant_2d(nx, ny, nx)
    U = U * (1.0 + 1e-2 * np.random.default_rng(ny).standard_normal(U.shape))
    res = []
    for rows in (0, 1, 3, 4, 5, 13, 20, 62):  # 0: the tile kernel
        say(f"[row] {nx}x{ny} {kw} rows={rows}")
        p = capi.params_default(nx, ny, 1, dx, bc=[1, 2, 0, 0, 1, 1], **kw)
        ctx = capi.Context(nx, ny, 1, dx, 1.4, p)
        ctx.tune(zchunk=rows)
        A = to_dev(U)
        D = torch.full_like(A, float("nan"))
        ctx.rhs(A, D)
        ctx.advance(A, 3, 1e300)
        torch.cuda.synchronize()
        assert ctx.status() == 0
        res.append((to_host(D), to_host(A), ctx.clock()))
        ctx.close()
    for r in res[1:]:
        assert np.array_equal(r[0], res[0][0])
        assert np.array_equal(r[1], res[0][1])
        assert r[2] == res[0][2]
