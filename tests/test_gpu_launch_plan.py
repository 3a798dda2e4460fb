"""The launch shapes that tuning leaves behind."""
import numpy as np
import pytest
import torch

from paper_2411_03090_amd import lks, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


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
