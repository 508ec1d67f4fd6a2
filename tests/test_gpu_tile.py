"""2D tile kernel (a stage and its corrections in one launch) against the row
kernel and its correction kernels."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say, to_dev, to_host
from paper_1908_02464_amd import workloads as w

pytestmark = pytest.mark.gpu
G = 1.4


@pytest.fixture(scope="module")
def capi():
    from paper_1908_02464_amd import capi as c
    c.lib()
    return c


def _noisy(nx, ny, seed):
    U, dx, _ = w.four_quadrant_2d(nx, ny, seed)
    return U * (1.0 + 1e-3 * np.random.default_rng(seed).standard_normal(U.shape)), dx


# edges of the 63-column tiles and of the one- and three-row ones (a small grid
# takes one row per workgroup), each boundary rule and scheme, and grids whose
# last tile holds one column or one row
@pytest.mark.parametrize("nx,ny,bc,kw", [
    (3, 2, [0, 0, 0, 0], {}), (63, 4, [1, 1, 2, 1], {}), (64, 3, [2, 2, 0, 0], {"split": 2}),
    (67, 45, [1, 1, 1, 1], {}), (126, 7, [0, 0, 2, 2], {"hybrid": 1}), (127, 200, [1, 2, 1, 1], {}),
    (190, 301, [0, 0, 0, 0], {"split": 1}), (253, 152, [2, 1, 1, 2], {"split": 1, "hybrid": 2, "weights": 2}),
    (316, 100, [1, 1, 0, 0], {"hybrid": 2}), (400, 130, [1, 1, 1, 1], {"hybrid": 3}),
    (128, 199, [0, 0, 1, 2], {"split": 2, "hybrid": 2, "weights": 1})])
def test_tile_bitwise(capi, nx, ny, bc, kw):
    """dU/dt and four advance() steps (global LF: the speeds folded by the
    stage before) carry the bits of the row kernel."""
    import torch
    say(f"[tile] {nx}x{ny} bc={bc} {kw}")
    U, dx = _noisy(nx, ny, nx + ny)
    res = []
    for rows in (0, 4):
        ctx = capi.Context(nx, ny, 1, dx, G, capi.params_default(nx, ny, 1, dx, bc=bc + [1, 1], **kw))
        ctx.tune(zchunk=rows)  # 0: the tile kernel; rows per item: the row kernel
        A = to_dev(U)
        D = torch.full_like(A, float("nan"))
        ctx.rhs(A, D)
        ctx.advance(A, 4, 1e300)
        torch.cuda.synchronize()
        assert ctx.status() == 0 and ctx.clock()[2] == 4
        res.append((to_host(D), to_host(A), ctx.clock()))
        ctx.close()
    assert np.array_equal(res[0][0], res[1][0])
    assert np.array_equal(res[0][1], res[1][1])
    assert res[0][2] == res[1][2]


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("nx", [128, 512])
def test_tile_state_sides_bitwise(capi, nx, split):
    """Inflow and state sides formed in the tile kernel (the moving front at
    each stage's time), a call of several steps clipped by t_end."""
    import torch
    U, dx, kw, inflow = w.double_mach(nx, nx // 4)
    kw["split"] = split
    te = 5.5 * (0.02 / (nx // 4))
    res = []
    for rows in (0, 3):
        ctx = capi.Context(nx, nx // 4, 1, dx, G, capi.params_default(nx, nx // 4, 1, dx, **kw))
        ctx.set_inflow(to_dev(inflow))
        ctx.tune(zchunk=rows)
        A = to_dev(U)
        D = torch.empty_like(A)
        ctx.rhs(A, D)
        ctx.advance(A, 5, te)
        ctx.advance(A, 20, te)
        torch.cuda.synchronize()
        assert ctx.status() == 0
        res.append((to_host(D), to_host(A), ctx.clock()))
        ctx.close()
    assert np.array_equal(res[0][0], res[1][0])
    assert np.array_equal(res[0][1], res[1][1])
    assert res[0][2] == res[1][2]
