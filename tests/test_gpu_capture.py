"""Calls of a context captured into a graph: every replay, with eager work in
between, gives what the same call gives eagerly, and so does an eager call after
the replays."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say
from paper_1908_02464_amd import workloads as w

pytestmark = pytest.mark.gpu
G = 1.4


@pytest.fixture(scope="module")
def capi():
    from paper_1908_02464_amd import capi as c
    c.lib()
    return c


def _state(shape):
    nx, ny, nz = shape
    if nz > 1:
        U, dx = w.turbulence_3d(nx, 5, ny=ny, nz=nz)
        U = U.copy()
        U[0, :, :, : nx // 2] *= 2.0
        U[4, :, :, : nx // 2] *= 2.0
        return U, dx
    if ny > 1:
        return w.four_quadrant_2d(nx, ny, 11)[:2]
    return w.shu_osher(nx)


# 1D: whole steps in one launch and in one per step, stages with lists (LF); 2D:
# tile kernel, row kernel with per-cell and face-once corrections; 3D: face
# lists, every face WENO; odd and even numbers of stages in the graph
@pytest.mark.parametrize("shape,rows,kw", [
    ((300, 1, 1), 0, {}), ((900, 1, 1), 0, {"hybrid": 2}), ((900, 1, 1), 0, {"split": 1, "hybrid": 2}),
    ((67, 45, 1), 0, {"split": 1}), ((67, 45, 1), 5, {"hybrid": 2}), ((400, 350, 1), 7, {"split": 1}),
    ((24, 20, 18), 0, {}), ((24, 20, 18), 0, {"hybrid": 2, "split": 1})])
@pytest.mark.parametrize("mode,n", [("rhs", 1), ("step", 1), ("step", 2), ("advance", 3)])
def test_replays_equal_eager_calls(capi, shape, rows, kw, mode, n):
    import torch
    U, dx = _state(shape)
    bc = [0] * 6 if shape[2] > 1 else [1] * 6
    p = capi.params_default(*shape, dx, bc=bc, **kw)
    st = torch.cuda.Stream()
    U = torch.from_numpy(np.ascontiguousarray(U)).cuda()

    def call(ctx, A, D):
        if mode == "rhs":
            ctx.rhs(A, D)
            with torch.cuda.stream(st):
                A.mul_(1.001)  # another state for the next replay
        elif mode == "step":
            for _ in range(n):
                ctx.step(A)
        else:
            ctx.advance(A, n, 1e300)

    def make():
        ctx = capi.Context(*shape, dx, G, p, stream=st)
        ctx.tune(zchunk=rows)
        A, D = U.clone(), torch.zeros_like(U)
        torch.cuda.synchronize()
        return ctx, A, D

    say(f"[capture] {shape} rows={rows} {kw} {mode} x{n}: eager")
    ctx, A, D = make()
    ref = []
    for _ in range(5):
        call(ctx, A, D)
        st.synchronize()
        ref.append((A.clone(), D.clone()))
    torch.cuda.synchronize()
    ctx.close()
    ctx, A, D = make()
    call(ctx, A, D)  # one eager call, then the capture
    st.synchronize()
    assert torch.equal(A, ref[0][0]) and torch.equal(D, ref[0][1])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        call(ctx, A, D)
    for k in range(1, 4):
        say(f"[capture]   replay {k}")
        with torch.cuda.stream(st):
            g.replay()
        st.synchronize()
        torch.ones(1 << 18, device="cuda").cumsum(0)
        torch.cuda.synchronize()
        assert torch.equal(A, ref[k][0]) and torch.equal(D, ref[k][1]), k
    call(ctx, A, D)
    torch.cuda.synchronize()
    assert torch.equal(A, ref[4][0]) and torch.equal(D, ref[4][1])
    ctx.close()
