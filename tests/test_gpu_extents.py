"""Grids at the ends of the accepted shapes, on the device."""
from __future__ import annotations

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
G = 1.4


def _flow(nx, ny):
    """A 2D state made on the device: jumps and noise over the whole grid."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    U = torch.empty((4, 1, ny, nx), dtype=torch.float64, device="cuda")
    n = nx * ny
    rho = 1.0 + 0.5 * ((torch.arange(n, device="cuda") // 7) % 3).double() + 0.1 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    U[0] = rho.view(1, ny, nx)
    for k in (1, 2):
        U[k] = (rho * (0.2 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64) - 0.1)).view(1, ny, nx)
    U[3] = (2.5 * rho + 0.5 * (U[1] ** 2 + U[2] ** 2).view(-1) / rho).view(1, ny, nx)
    return U


def test_more_tiles_than_a_launch_holds():
    """A narrow grid of 10 M tiles (two launches per stage): the bits of the
    row kernel and its corrections."""
    import torch
    from paper_1908_02464_amd import capi
    nx, ny = 2, 30_000_001
    say(f"[extents] {nx}x{ny}")
    U = _flow(nx, ny)
    p = capi.params_default(nx, ny, 1, 1.0, bc=[0, 0, 1, 2, 1, 1], hybrid=2)
    ctx = capi.Context(nx, ny, 1, 1.0, G, p)
    D = [torch.full_like(U, float("nan")) for _ in range(2)]
    for rows, d in zip((0, 20), D):
        ctx.tune(zchunk=rows)
        ctx.rhs(U, d)
        torch.cuda.synchronize()
    ctx.close()
    assert bool(torch.isfinite(D[0]).all()) and float(D[0].abs().max()) > 0.1
    assert torch.equal(D[0], D[1])


def test_columns_past_32_bit_offsets():
    """A 2D grid wider than 2^29 columns (2^32 bytes a row): dU/dt around the
    columns where a 32-bit byte offset would wrap, and at both ends, carries
    the bits of small grids cut out there."""
    import torch
    from paper_1908_02464_amd import capi
    nx, ny = (1 << 29) + 500, 2
    need = nx * ny * 8 * 4 * 2 + nx * ny * (3 * 32 + 8 + 68)  # U, dU/dt and the context
    free, _ = torch.cuda.mem_get_info()
    if free < need + (8 << 30):
        pytest.skip(f"{free >> 30} GiB of device memory free, {need >> 30} needed")
    say(f"[extents] {nx}x{ny}: {need >> 30} GiB")
    U = torch.empty((4, 1, ny, nx), dtype=torch.float64, device="cuda")
    step = 1 << 26
    for x in range(0, nx, step):
        n = min(step, nx - x)
        U[:, :, :, x:x + n] = _flow(n, ny)
    torch.cuda.empty_cache()
    D = torch.full_like(U, float("nan"))
    p = capi.params_default(nx, ny, 1, 1.0, bc=[1, 1, 0, 0, 1, 1])
    ctx = capi.Context(nx, ny, 1, 1.0, G, p)
    ctx.rhs(U, D)
    torch.cuda.synchronize()
    ctx.close()
    w = 200
    for x in (0, (1 << 28) - 100, (1 << 29) - 100, nx - w):
        V = U[:, :, :, x:x + w].contiguous()
        q = capi.params_default(w, ny, 1, 1.0, bc=[1, 1, 0, 0, 1, 1], thr_L=(p.thr_L[0], p.thr_L[1], 1.0))
        E = torch.empty_like(V)
        c = capi.Context(w, ny, 1, 1.0, G, q)
        c.rhs(V, E)
        torch.cuda.synchronize()
        c.close()
        a, b = 0 if x == 0 else 3, w if x == nx - w else w - 3  # cells whose stencils lie in the cut
        assert float(E.abs().max()) > 0.01
        assert torch.equal(D[:, :, :, x + a:x + b], E[:, :, :, a:b]), x
    del U, D, V, E
    torch.cuda.empty_cache()
