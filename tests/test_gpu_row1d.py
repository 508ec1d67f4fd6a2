"""1D corrections by the stage kernels (step(), the right-hand side) on either
side of the size from which their kernel runs three wavefronts per SIMD."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import say, to_dev, to_host
from paper_1908_02464_amd import workloads as w

pytestmark = pytest.mark.gpu


# 131072 cells, one more, and enough that a lane takes several cells
@pytest.mark.parametrize("n", [131072, 131073, 600001])
@pytest.mark.parametrize("kw", [{"hybrid": 2}, {"hybrid": 2, "split": 1, "weights": 2}, {"hybrid": 1, "split": 2}])
def test_long_lists_1d(n, kw):
    """dU/dt against the per-direction sweeps: in units of the state after one
    CFL step within 1e-12, the bar of the sweeps elsewhere."""
    import torch
    from gpu_util import rhs_err
    from paper_1908_02464_amd import capi
    say(f"[row 1d] n={n} {kw}")
    U, dx = w.shu_osher(n)
    U = U * (1.0 + 1e-3 * np.random.default_rng(n).standard_normal(U.shape))
    D = []
    for path in (capi.PATH_AUTO, capi.PATH_SWEEPS):
        ctx = capi.Context(n, 1, 1, dx, 1.4, capi.params_default(n, 1, 1, dx, bc=[1, 2, 1, 1, 1, 1], **kw))
        ctx.tune(path)
        A = to_dev(U)
        d = torch.full_like(A, float("nan"))
        ctx.rhs(A, d)
        dt, st = ctx.cfl_dt(A)
        torch.cuda.synchronize()
        assert st == 0
        D.append(to_host(d))
        ctx.close()
    assert np.all(np.isfinite(D[0]))
    err = rhs_err(D[0], D[1], U, dt)
    say(f"    err = {err:.2e}")
    assert err <= 1e-12
