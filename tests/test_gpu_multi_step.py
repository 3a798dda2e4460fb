"""Several steps per launch (the kernels small grids take by default) against
one step per launch of the tile kernels: the same states, adjoint fields and
sensitivities bit for bit, objectives to the rounding of their sum. The grids
sit at the edges of the launch shapes: a few nodes wide, one tile, tiles next
to all four corners, more tiles than the tile kernels have accumulators, each
block size, several rounds of blocks; the step counts leave remainders."""
import numpy as np
import pytest
import torch

from paper_2411_03090_amd import lks, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def T(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float64).reshape(-1), device=DEV)


def _run(wl, prec, tiles, ckpt=None, budget=0):
    c = lks.LKS(wl, precision=prec, device=DEV, checkpointing=ckpt, mem_budget=budget)
    if tiles:
        c.set_tile_rows(4)
        c.set_steps_per_launch(1, 1)
    g = T(wl.gamma)
    dJ = torch.full_like(g, float("nan"))
    c.forward(g, wl.n_fwd)
    J = c.objective()
    names = ["drho", "ux", "uy"] + (["T"] if wl.thermal else [])
    out = {n: c.read(n).cpu().numpy() for n in names}
    c.backward(1.0, dJ, wl.n_adj)
    names = ["adj_rho", "adj_vx", "adj_vy"] + (["adj_theta"] if wl.thermal else [])
    out.update({n: c.read(n).cpu().numpy() for n in names})
    out["dJ"] = dJ.cpu().numpy()
    return J, out


def _same(wl, prec, **kw):
    print(f"[gpu] {wl.name} {prec} {wl.n_fwd}+{wl.n_adj} {kw}", flush=True)
    J0, a = _run(wl, prec, True, **kw)
    J1, b = _run(wl, prec, False, **kw)
    # the objective sums the same terms in another order: a few units in the
    # last place of the largest partial sum
    assert abs(J1 - J0) <= 1e-13 * max(abs(J0), 1e-3), (J0, J1)
    for n in a:
        assert np.array_equal(a[n], b[n]), n
        assert np.isfinite(b[n]).all()


@pytest.mark.parametrize("prec", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,n,m", [(4, 4, 1, 1), (5, 4, 13, 8), (64, 64, 29, 31),
                                       (131, 9, 20, 7), (201, 150, 15, 16),
                                       (333, 217, 12, 11), (700, 500, 9, 10)])
def test_steady(nx, ny, n, m, prec):
    _same(W.steady_channel_uniform(nx, ny, seed=3, n_fwd=n, n_adj=m), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,n,m", [(1251, 1000, 1, 1), (1800, 1670, 7, 8), (128, 9800, 6, 7),
                                       (129, 23300, 5, 4), (9801, 129, 8, 7)])
def test_steady_large(nx, ny, n, m, prec):
    """The marching kernels: odd sides, strips whose last lanes lie off the grid,
    two strips, chunks of a few rows, remainders of two and three steps."""
    _same(W.steady_channel_uniform(nx, ny, seed=3, n_fwd=n, n_adj=m), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [7, 70, 201])
def test_heat_source(n, prec):
    _same(W.heat_exchanger(n=n, n_fwd=23, n_adj=22, sigma=2.0), prec)


@pytest.mark.parametrize("mode", ["paper", "exact"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", [(41, 37), (141, 161), (390, 301)])
def test_heat_sink(nx, ny, prec, mode):
    wl = W.heat_sink(nx=nx, ny=ny, n_steps=33, sigma=3.0)
    wl.adjoint_mode = mode
    _same(wl, prec)


@pytest.mark.parametrize("mode", ["paper", "exact"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("plan", ["all", "two_level", "binomial"])
def test_unsteady_channel_plans(plan, prec, mode):
    wl = W.unsteady_thermal_channel(70, 26, Re=60.0, sigma=3.0, seed=4, n_steps=61, period=40.0)
    wl.mask = W.channel_mask(70, 26, thermal=True, probe_col=20)
    wl.adjoint_mode = mode
    r = 8 if prec == "fp64" else 4
    kw = {"all": {}, "two_level": {"budget": 70 * 26 * r * (4 * 16 + 60)},
          "binomial": {"ckpt": ("binomial", 5)}}[plan]
    _same(wl, prec, **kw)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (70, 26), (128, 33)])
def test_periodic_box(nx, ny, prec):
    wl = W.periodic_box(nx, ny, nu=0.08, thermal=True)
    wl.gamma = W.gamma_grf(nx, ny, 2.0, 5)
    wl.alpha_max, wl.beta_max, wl.objective = 1.0, 0.1, W.OBJ_HEAT_EXCHANGE
    wl.gbeta, wl.T_ref = (0.0, 1e-4), 0.5
    wl.mode, wl.n_fwd, wl.n_adj, wl.ufac = W.MODE_UNSTEADY, 19, 19, np.ones(20)
    _same(wl, prec)


def _batch(wls, prec, rows, n, m, **kw):
    b = lks.Batch(wls, precision=prec, device=DEV, **kw)
    if rows:
        b.set_tile_rows(rows)
    gs = [T(w.gamma) for w in wls]
    outs = [torch.full_like(g, float("nan")) for g in gs]
    runs = []
    for graph in (True, True, False):  # captured, replayed, eager
        J = b.run(gs, outs, n, m, graph=graph)
        names = ["adj_rho", "adj_vx", "adj_vy"] + (["adj_theta"] if wls[0].thermal else [])
        if wls[0].mode == W.MODE_STEADY:
            names += ["drho", "ux", "uy"]
        fields = [b.read(d, f).cpu().numpy() for d in range(len(wls)) for f in names]
        runs.append((J, [o.cpu().numpy() for o in outs] + fields))
    for J, x in runs[1:]:
        assert J == runs[0][0]
        assert all(np.array_equal(p, q) for p, q in zip(x, runs[0][1]))
    return runs[0]


# the first batch fits one round of the smallest tiles, the second takes the
# tiles of several rounds; MARCHED take the marching kernels (the first in FP32 only)
BATCHES = [[(31, 31), (5, 4), (64, 40)], [(150, 131), (512, 300), (700, 513)]]


MARCHED = [[(5, 4), (1100, 900), (64, 65), (65, 9), (700, 701)],
           [(5, 4), (1400, 1100)], [(257, 1030), (1700, 1600), (130, 120), (4, 30)]]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", BATCHES + MARCHED)
def test_steady_batch(sizes, prec):
    wls = [W.steady_channel_uniform(x, y, Re=20.0, seed=d, n_fwd=11, n_adj=10)
           for d, (x, y) in enumerate(sizes)]
    print(f"[gpu] steady batch {sizes} {prec}", flush=True)
    J0, a = _batch(wls, prec, 4, 11, 10)
    J1, b = _batch(wls, prec, None, 11, 10)
    assert J0 == J1
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("mode", ["paper", "exact"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", BATCHES)
def test_unsteady_batch(sizes, prec, mode):
    n = 23
    wls = []
    for d, (x, y) in enumerate(sizes):
        w = W.unsteady_thermal_channel(x, y, Re=60.0, sigma=3.0, seed=d, n_steps=n, period=9.0)
        w.mask = W.channel_mask(x, y, thermal=True, probe_col=2)
        wls.append(w)
    full = lks.Batch(wls, precision=prec, bind=False)
    r = 8 if prec == "fp64" else 4
    # room for about half of the levels: checkpoints and replayed segments
    budget = full.workspace_size() - int(0.5 * n * 3 * r * sum(w.n_nodes for w in wls))
    print(f"[gpu] unsteady batch {sizes} {prec} {mode}", flush=True)
    kw = dict(mem_budget=budget, adjoint_mode=mode)
    J0, a = _batch(wls, prec, 4, n, n, **kw)
    J1, b = _batch(wls, prec, None, n, n, **kw)
    # the objective sums the same terms in another order
    assert all(abs(x - y) <= 1e-13 * max(abs(x), 1e-3) for x, y in zip(J0, J1))
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
