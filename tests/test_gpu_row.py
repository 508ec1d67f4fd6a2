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


# global LF: the speeds folded by the stage before (row kernel and its
# corrections: face once from 131072 cells, else per cell) against one step per
# call, which reduces them from the state
@pytest.mark.parametrize("nx,ny,rows,hybrid", [(130, 67, 5, 0), (400, 350, 7, 0), (400, 350, 7, 2), (900, 760, 0, 0)])
def test_row_folded_lf_speeds(nx, ny, rows, hybrid):
    import torch
    from paper_1908_02464_amd import capi
    say(f"[row] LF {nx}x{ny} rows={rows} hybrid={hybrid}")
    U, dx, _ = w.four_quadrant_2d(nx, ny, nx)
    res = []
    for one_call in (True, False):
        p = capi.params_default(nx, ny, 1, dx, bc=[1, 1, 0, 0, 1, 1], split=1, hybrid=hybrid)
        ctx = capi.Context(nx, ny, 1, dx, 1.4, p)
        ctx.tune(zchunk=rows)
        A = to_dev(U)
        if one_call:
            ctx.advance(A, 4, 1e300)
        else:
            for _ in range(4):
                ctx.step(A)
        torch.cuda.synchronize()
        assert ctx.status() == 0
        res.append(to_host(A))
        ctx.close()
    assert np.array_equal(res[0], res[1])
