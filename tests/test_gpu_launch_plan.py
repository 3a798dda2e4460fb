"""The launch shapes that tuning leaves behind, and the several-steps kernels of
batches at every launch shape they choose among."""
import numpy as np
import pytest
import torch

from paper_2411_03090_amd import lks, workloads as W
from test_gpu_multi_step import _batch
from test_launch_plan import CANDIDATES

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def unsteady_channel(nx, ny, n, seed=0):
    """Channel without temperature, oscillating inflow, pressure drop averaged over
    n steps."""
    wl = W.steady_channel_uniform(nx, ny, Re=20.0, seed=seed, n_fwd=n, n_adj=n)
    wl.mode = W.MODE_UNSTEADY
    wl.ufac = 1.0 + 0.5 * np.sin(2.0 * np.pi * np.arange(n + 1) / 9.0)
    return wl


def T(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float64).reshape(-1), device=DEV)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_tuning_times_the_kernels_that_were_turned_off(precision):
    """A tile height set before, by the caller or by an earlier tuning, does not
    hide the several-steps kernels, three times as fast on 64 x 64, from the
    tuner."""
    wl = W.steady_channel_uniform(64, 64, n_fwd=4, n_adj=4)
    c = lks.LKS(wl, precision=precision, device=DEV)
    plan = c.launch_plan()
    assert plan[0][0] == plan[1][0] == "multi"
    c.set_tile_rows(4)
    assert c.launch_plan()[0][0] == "tile"
    c.autotune(T(wl.gamma), 200)
    assert c.launch_plan() == plan


def test_batch_tuning_times_the_kernels_that_were_turned_off():
    """Three 900 x 900 designs march 1.3 times as fast as their tiles run."""
    wls = [W.steady_channel_uniform(900, 900, seed=d, n_fwd=4, n_adj=4) for d in range(3)]
    b = lks.Batch(wls, precision="fp32", device=DEV)
    plan = b.launch_plan()
    assert plan == ("march", 2, 2)
    b.set_tile_rows(8)
    gs = [T(w.gamma) for w in wls]
    b.autotune(gs, [torch.empty_like(g) for g in gs], 100)
    assert b.launch_plan() == plan


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", [c[0] for c in CANDIDATES])
def test_steady_batch_candidates(sizes, precision):
    """Each candidate of the several-steps batches against the tile kernels, bit
    for bit, with step counts that leave remainders."""
    wls = [W.steady_channel_uniform(x, y, Re=20.0, seed=d, n_fwd=11, n_adj=10)
           for d, (x, y) in enumerate(sizes)]
    print(f"[gpu] steady batch {len(sizes)} x {sizes[0]} {precision}", flush=True)
    assert lks.Batch(wls, precision=precision, bind=False).launch_plan()[0] == "multi"
    J0, a = _batch(wls, precision, 4, 11, 10)
    J1, b = _batch(wls, precision, None, 11, 10)
    assert J0 == J1
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("thermal,mode", [(True, "paper"), (True, "exact"), (False, "paper")])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", [c[0] for c in CANDIDATES])
def test_unsteady_batch_candidates(sizes, precision, thermal, mode):
    """The same with checkpoints and replays; the objective sums the same terms in
    another order: some units in the last place of the largest partial sum, which
    the sums of 23 levels of densities of below 1, averaged, leave below 1e-13."""
    n, wls = 23, []
    for d, (x, y) in enumerate(sizes):
        if thermal:
            w = W.unsteady_thermal_channel(x, y, Re=60.0, sigma=3.0, seed=d, n_steps=n, period=9.0)
            w.mask = W.channel_mask(x, y, thermal=True, probe_col=2)
        else:
            w = unsteady_channel(x, y, n, seed=d)
        wls.append(w)
    full = lks.Batch(wls, precision=precision, bind=False)
    assert full.launch_plan()[0] == "multi"
    r = 8 if precision == "fp64" else 4
    # room for about half of the levels
    budget = full.workspace_size() - int(0.5 * n * (3 if thermal else 2) * r
                                         * sum(w.n_nodes for w in wls))
    print(f"[gpu] unsteady batch {len(sizes)} x {sizes[0]} {precision} {thermal} {mode}",
          flush=True)
    kw = dict(mem_budget=budget, adjoint_mode=mode)
    J0, a = _batch(wls, precision, 4, n, n, **kw)
    J1, b = _batch(wls, precision, None, n, n, **kw)
    assert all(abs(x - y) <= 1e-13 * max(abs(x), 1.0) for x, y in zip(J0, J1))
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


def test_a_batch_bound_again_captures_its_steps_again():
    """The captured sequence holds addresses of the workspace it was captured on."""
    wls = [W.steady_channel_uniform(40, 24, Re=20.0, seed=d, n_fwd=9, n_adj=8) for d in range(2)]
    b = lks.Batch(wls, precision="fp64", device=DEV)
    gs = [T(w.gamma) for w in wls]
    outs = [torch.empty_like(g) for g in gs]
    J0 = b.run(gs, outs, 9, 8)
    ref = [o.clone() for o in outs]
    first = b.workspace  # kept: the sequence of before would still run on it
    b.bind()
    first.zero_()
    for o in outs:
        o.zero_()
    assert b.run(gs, outs, 9, 8) == J0
    assert all(torch.equal(o, r) for o, r in zip(outs, ref))
    assert not first.any()
