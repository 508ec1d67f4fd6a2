"""The time step of a context whose advance() has stopped (at t_end, or at a
non-physical state): step() and cfl_dt() take it from the state they are given
and from nothing that the stopped call left behind."""
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


def _state(shape, u, p):
    """Uniform density and pressure, the halves along x moving apart (u > 0)."""
    nx, ny, nz = shape
    x = np.arange(nx) < nx // 2
    ux = np.broadcast_to(np.where(x, -u, u), (nz, ny, nx))
    vel = [ux, np.zeros_like(ux), np.zeros_like(ux)][: 1 + (ny > 1) + (nz > 1)]
    return w.conserved(np.ones((nz, ny, nx)), vel, np.full((nz, ny, nx), p))


# the tile kernel (one row and three rows per workgroup, global LF, every face
# WENO), the row kernel with its corrections per cell and face once, the 1D and
# the 3D kernels
CASES = [((67, 45, 1), 0, {}), ((400, 300, 1), 0, {}), ((400, 300, 1), 0, {"split": 1}),
         ((200, 130, 1), 0, {"hybrid": 2}), ((67, 45, 1), 4, {}), ((400, 350, 1), 7, {"split": 1}),
         ((300, 1, 1), 0, {}), ((900, 1, 1), 0, {}), ((300, 1, 1), 0, {"split": 1}),
         ((20, 18, 17), 0, {}), ((20, 18, 17), 0, {"hybrid": 2})]


@pytest.mark.parametrize("stop", ["t_end", "nonphysical"])
@pytest.mark.parametrize("shape,rows,kw", CASES)
def test_time_step_after_a_stopped_call(capi, shape, rows, kw, stop):
    import torch
    say(f"[clock] {shape} rows={rows} {kw} stopped at {stop}")
    dx = 1.0 / max(shape)
    # a CFL number of 30 has the run end at a negative pressure or a NaN
    p = capi.params_default(*shape, dx, cfl=0.5 if stop == "t_end" else 30.0, **kw)
    slow = _state(shape, 0.1, 1.0)
    res = []
    for used in (True, False):
        ctx = capi.Context(*shape, dx, G, p)
        ctx.tune(zchunk=rows)
        if used:
            if stop == "t_end":  # fast state, more steps than reach t_end
                A = to_dev(_state(shape, 0.5, 50.0))
                ctx.advance(A, 12, 4.5 * 0.5 * dx / 20.0)
                assert ctx.status() == 0 and 1 < ctx.clock()[2] < 12
            else:
                A = to_dev(_state(shape, 2.0, 1.0))
                ctx.advance(A, 60, 1e300)
                assert ctx.status(clear=True) & 1 and 0 < ctx.clock()[2] < 60
        B = to_dev(slow)
        dt, st = ctx.cfl_dt(B)
        assert st == 0
        ctx.step(B)
        torch.cuda.synchronize()
        res.append((dt, ctx.time()[1], to_host(B)))
        if used:  # and once more, straight after another stopped call
            if stop == "t_end":
                A = to_dev(_state(shape, 0.5, 50.0))
                t = ctx.clock()[0]
                ctx.advance(A, 12, t + 4.5 * 0.5 * dx / 20.0)
                assert ctx.status() == 0
            else:
                A = to_dev(_state(shape, 2.0, 1.0))
                ctx.advance(A, 60, 1e300)
                assert ctx.status(clear=True) & 1
            C = to_dev(slow)
            ctx.step(C)
            torch.cuda.synchronize()
            res.append((dt, ctx.time()[1], to_host(C)))
        ctx.close()
    fresh = res[-1]
    assert fresh[0] == fresh[1] > 0.0
    for r in res[:-1]:
        assert r[:2] == fresh[:2]
        assert np.array_equal(r[2], fresh[2], equal_nan=True)
