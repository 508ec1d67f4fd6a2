"""1D whole-step kernels of advance() against the stage kernels (step())."""
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


# edges of the workgroup kernel (252 cells on four wavefronts, 504 on eight)
# and of the 46-cell tiles of the per-step kernel, each boundary rule, an even
# and an odd number of steps (the per-step kernel alternates two arrays)
@pytest.mark.parametrize("n,steps,bc,kw", [
    (5, 4, 0, {}), (252, 7, 2, {"split": 2}), (253, 6, 0, {"hybrid": 2}), (504, 5, 1, {}),
    (505, 4, 0, {}), (506, 5, 2, {"split": 2, "hybrid": 1}), (507, 3, 1, {"hybrid": 2, "weights": 2}),
    (551, 6, 2, {}), (553, 3, 0, {"hybrid": 2, "weights": 1}), (4700, 4, 1, {"hybrid": 3}),
    (600, 4, 3, {}), (70, 5, 3, {"split": 2})])
def test_line_steps_bitwise(capi, n, steps, bc, kw):
    """The same bits, clock and step count as step-by-step launches, in one
    call and in calls of one step each."""
    import torch
    say(f"[line] n={n} steps={steps} bc={bc} {kw}")
    left, right = w.SOD if n < 16 else w.random_two_state(np.random.default_rng(n))
    U, dx = w.riemann_1d(n, left, right)
    U = U * (1.0 + 1e-3 * np.random.default_rng(1).standard_normal(U.shape))  # faces flagged everywhere
    sides = [3, 1, 1, 1, 1, 1] if bc == 3 else [bc, bc, 1, 1, 1, 1]
    got = []
    for how in ("step", "one", "many"):
        ctx = capi.Context(n, 1, 1, dx, G, capi.params_default(n, 1, 1, dx, bc=sides, **kw))
        if bc == 3:
            ctx.set_inflow(to_dev(np.ascontiguousarray(U[:, 0, 0, :1] * 1.1)))
        A = to_dev(U)
        if how == "step":
            if bc == 3:  # step() bounds its dt by the inflow speed as advance() does
                for _ in range(steps):
                    ctx.step(A, ctx.cfl_dt(A)[0])
            else:
                for _ in range(steps):
                    ctx.step(A)
        elif how == "one":
            ctx.advance(A, steps, 1e300)
        else:
            for _ in range(steps):
                ctx.advance(A, 1, 1e300)
        torch.cuda.synchronize()
        if how != "step":
            t, _, k = ctx.clock()
            assert k == steps and ctx.status() == 0
            got.append((to_host(A), t))
        else:
            got.append((to_host(A), None))
        ctx.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][0], got[2][0])
    assert got[1][1] == got[2][1] > 0.0


@pytest.mark.parametrize("n", [300, 900])
@pytest.mark.parametrize("steps", [9, 10])
def test_line_stops_at_t_end(capi, n, steps):
    """A call with more steps than reach t_end: the last one is clipped, the
    rest pass the state on; a second call changes nothing."""
    import torch
    U, dx = w.sod(n)
    te = 5.5 * 0.5 * dx / 1.9
    ref = None
    for k in (steps, 40):
        ctx = capi.Context(n, 1, 1, dx)
        A = to_dev(U)
        ctx.set_time(0.0)
        ctx.advance(A, k, te)
        t, dt, taken = ctx.clock()
        assert t == te and taken < steps and dt == 0.0
        ctx.advance(A, 3, te)
        torch.cuda.synchronize()
        assert ctx.clock()[0] == te and ctx.clock()[2] == taken
        got = to_host(A)
        ctx.close()
        assert ref is None or np.array_equal(got, ref)
        ref = got
