"""Several steps per launch in unsteady sweeps without temperature: levels kept
inside a launch, the pressure drop summed per tile (on the small grid in the
accumulators behind the boundary operators), the adjoint with a moving state
and the unseeded level 0, under every checkpoint plan. The same bits as one step
per launch of the tile kernels, and the oracle's gradient."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2411_03090_amd import lks
from test_gpu_launch_plan import unsteady_channel
from test_gpu_multi_step import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("plan", ["all", "two_level", "binomial"])
@pytest.mark.parametrize("nx,ny,n,mode", [(70, 26, 61, "paper"), (70, 26, 61, "exact"),
                                          (333, 217, 25, "paper")])
def test_unsteady_pressure_drop(nx, ny, n, mode, plan, precision):
    wl = unsteady_channel(nx, ny, n, seed=5)
    wl.adjoint_mode = mode
    r = 8 if precision == "fp64" else 4
    c = lks.LKS(wl, precision=precision, bind=False)
    assert c.launch_plan()[0][0] == c.launch_plan()[1][0] == "multi"
    budget = c.workspace_size() - int(0.4 * n) * 2 * r * nx * ny
    kw = {"all": {}, "two_level": {"budget": budget, "ckpt": ("two_level", 0)},
          "binomial": {"ckpt": ("binomial", 4)}}[plan]
    print(f"[gpu] unsteady channel {nx}x{ny} {n} {mode} {plan} {precision}", flush=True)
    J0, a = _run(wl, precision, True, **kw)
    J1, b = _run(wl, precision, False, **kw)
    for f in a:
        assert np.array_equal(a[f], b[f]), f
        assert np.isfinite(b[f]).all()
    # the same terms in another order: some units in the last place of the
    # largest partial sum, averaged over the steps
    assert abs(J1 - J0) <= 1e-13 * max(abs(J0), 1.0)
    Jo, so, _, _ = O.gradient(wl)
    tol = 1e-12 if precision == "fp64" else 1e-3
    assert abs(J1 - Jo) <= tol * abs(Jo)
    assert np.linalg.norm(b["dJ"] - so.ravel()) <= tol * np.linalg.norm(so)
