"""Which kernels a context or batch takes can be read, and a launch shape can be
carried over to another context (planning only, no GPU)."""
import pytest

from paper_2411_03090_amd import lks, workloads as W


def _ctx(nx, ny, precision="fp32"):
    return lks.LKS(W.steady_channel_uniform(nx, ny, n_fwd=4, n_adj=4), precision=precision,
                   bind=False)


def _copy_shape(src, dst):
    """What a program that keeps launch shapes does with them."""
    ty, sf, sa = src.launch_shape()
    (kf, _), (ka, _) = src.launch_plan()
    dst.set_tile_rows(ty)
    dst.set_steps_per_launch(sf, sa)
    dst.set_launch_plan(kf, ka)


@pytest.mark.parametrize("nx,ny,precision,kernel", [
    (64, 64, "fp64", "multi"), (512, 512, "fp32", "multi"), (512, 512, "mixed", "multi"),
    (2048, 2048, "fp32", "march"), (2048, 2048, "fp64", "march"), (1024, 1024, "fp32", "tile")])
def test_plan_is_reported_and_restored(nx, ny, precision, kernel):
    a = _ctx(nx, ny, precision)
    (kf, sf), (ka, sa) = plan = a.launch_plan()
    assert kf == ka == kernel
    assert (sf > 1 and sa > 1) if kernel != "tile" else (sf, sa) == (1, 1)
    b = _ctx(nx, ny, precision)
    b.set_tile_rows(4)
    assert b.launch_plan() == (("tile", 1), ("tile", 1))
    b.set_steps_per_launch(2, 1)
    assert b.launch_plan() == (("tile", 2), ("tile", 1))
    _copy_shape(a, b)
    assert b.launch_plan() == plan and b.launch_shape() == a.launch_shape()
    b.set_launch_plan("tile", ka)
    assert b.launch_plan() == (("tile", 1), (ka, sa))


def test_refused_plans_change_nothing():
    a = _ctx(64, 64)
    plan = a.launch_plan()
    for fwd, adj in (("march", "multi"), ("multi", "march")):
        with pytest.raises(lks.LKSError) as e:
            a.set_launch_plan(fwd, adj)
        assert e.value.status == lks.LKS_E_UNSUPPORTED
    with pytest.raises(lks.LKSError) as e:
        lks._check(lks._lib.lks_set_launch_plan(a.ctx, 0, 3), a.ctx)
    assert e.value.status == lks.LKS_E_INVALID
    assert a.launch_plan() == plan
    d = lks.LKS(W.heated_block_duct(16, 8, 8, Re=20.0, n_steps=10), precision="fp32", bind=False)
    assert d.launch_plan() == (("tile", 1), ("tile", 1))
    with pytest.raises(lks.LKSError):
        d.set_launch_plan("multi", "tile")


def test_unsteady_plans():
    wl = W.unsteady_thermal_channel(64, 48, n_steps=50)
    c = lks.LKS(wl, precision="fp32", bind=False)
    (kf, sf), (ka, sa) = c.launch_plan()
    assert (kf, ka) == ("multi", "multi") and sf > 1 and sa > 1
    c.set_checkpointing("binomial", 4)  # whose reversal takes its adjoint steps one by one
    assert c.launch_plan() == ((kf, sf), ("tile", 1))


def test_batch_plan_is_reported_and_restored():
    wls = [W.steady_channel_uniform(512, 400, seed=d, n_fwd=4, n_adj=4) for d in range(16)]
    b = lks.Batch(wls, precision="fp32", bind=False)
    plan = b.launch_plan()
    assert plan == ("march", 2, 2)
    b.set_tile_rows(8)
    assert b.launch_plan() == ("tile", 1, 1)
    with pytest.raises(lks.LKSError) as e:
        b.set_launch_plan("multi")
    assert e.value.status == lks.LKS_E_UNSUPPORTED and b.launch_plan() == ("tile", 1, 1)
    b.set_launch_plan("march")
    assert b.launch_plan() == plan


def test_refused_shapes_change_nothing_in_a_mixed_context():
    """The FP32 part takes 16 rows, the FP64 part does not; FP64 thermal sweeps
    run one step per launch, FP32 ones two."""
    a = _ctx(512, 512, "mixed")
    plan = a.launch_plan()
    with pytest.raises(lks.LKSError):
        a.set_tile_rows(16)
    assert a.launch_plan() == plan
    b = lks.LKS(W.heat_exchanger(n=64, n_fwd=4, n_adj=4), precision="mixed", bind=False)
    plan = b.launch_plan()
    for steps in ((2, 2), (1, 3), (3, 1)):
        with pytest.raises(lks.LKSError):
            b.set_steps_per_launch(*steps)
        assert b.launch_plan() == plan
    b.set_steps_per_launch(1, 2)
    assert b.launch_plan() == (("tile", 1), ("tile", 2))


def _designs(sizes, thermal):
    if thermal:
        return [W.unsteady_thermal_channel(x, y, Re=60.0, seed=d, n_steps=9)
                for d, (x, y) in enumerate(sizes)]
    return [W.steady_channel_uniform(x, y, seed=d, n_fwd=4, n_adj=4)
            for d, (x, y) in enumerate(sizes)]


# (designs, FP32 steps per launch, FP64, FP64 thermal): each candidate of the
# batches that fit one round of blocks, and the last one, over several rounds
CANDIDATES = [
    ([(64, 64)] * 2, 6, 6, 6), ([(64, 64)] * 4, 6, 6, 6), ([(64, 64)] * 6, 5, 5, 5),
    ([(31, 31), (5, 4), (64, 40)], 6, 6, 6), ([(64, 64)] * 8, 4, 4, 4),
    ([(100, 100)] * 2, 5, 5, 5), ([(128, 128)] * 2, 5, 5, 5), ([(48, 48)] * 8, 5, 5, 5),
    ([(144, 144)] * 4, 6, 6, 3), ([(128, 128)] * 5, 6, 5, 3), ([(128, 128)] * 7, 5, 5, 2),
    ([(200, 200)] * 4, 4, 4, 2), ([(200, 200)] * 5, 3, 3, 2), ([(200, 200)] * 8, 2, 3, 2)]


@pytest.mark.parametrize("thermal", [False, True])
@pytest.mark.parametrize("sizes,f32,f64,f64t", CANDIDATES)
def test_small_batches_run_several_steps_per_launch(sizes, f32, f64, f64t, thermal):
    for precision, k in (("fp32", f32), ("fp64", f64t if thermal else f64)):
        b = lks.Batch(_designs(sizes, thermal), precision=precision, bind=False)
        assert b.launch_plan() == ("multi", k, k), precision


@pytest.mark.parametrize("thermal", [False, True])
def test_batch_budget_too_small_for_the_plans_table(thermal):
    """Four designs of 64 x 64 run 6 steps per launch on 256 tiles; the table of
    the tile kernels holds 64, which leave 4 steps. What a batch without the
    larger table needs is still enough."""
    wls = _designs([(64, 64)] * 4, thermal)
    b = lks.Batch(wls, precision="fp32", bind=False)
    full = b.workspace_size()
    b.set_memory_budget(full)
    assert b.launch_plan() == ("multi", 6, 6)
    small = lks.Batch(wls, precision="fp32", bind=False)
    # (unsteady: of the largest plan; its smaller ones fit with either table)
    tables = 8 * (256 - 64)
    if thermal:
        lo, hi = 1, full
        while hi - lo > 256:  # the smallest budget
            mid = (lo + hi) // 2
            try:
                lks.Batch(wls, precision="fp32", bind=False).set_memory_budget(mid)
                hi = mid
            except lks.LKSError:
                lo = mid
        small.set_memory_budget(hi)
    else:
        small.set_memory_budget(full - tables)
    assert small.launch_plan() == ("multi", 4, 4)
    with pytest.raises(lks.LKSError) as e:
        b.set_memory_budget(1)
    assert e.value.status == lks.LKS_E_NOMEM and b.launch_plan() == ("multi", 6, 6)
    assert b.workspace_size() == full
    b.set_tile_rows(8)
    with pytest.raises(lks.LKSError):
        b.set_memory_budget(1)
    assert b.launch_plan() == ("tile", 1, 1)


@pytest.mark.parametrize("sizes,thermal,f32,f64", [
    ([(256, 256)] * 5, False, "multi", "multi"), ([(200, 200)] * 24, False, "multi", "multi"),
    ([(1000, 1000)], False, "tile", "multi"), ([(300, 40)] * 30, False, "tile", "multi"),
    ([(1000, 10)] * 16, False, "multi", "tile"), ([(64, 64)] * 100, False, "multi", "multi"),
    ([(256, 256)] * 5, True, "multi", "multi"), ([(1000, 1000)], True, "multi", "multi"),
    ([(700, 5)] * 20, True, "tile", "tile"), ([(1000, 10)] * 16, True, "tile", "multi"),
    ([(5, 700)] * 20, True, "multi", "multi")])
def test_batches_of_several_rounds_take_the_faster_kernels(sizes, thermal, f32, f64):
    """Where several rounds of blocks were measured slower than the tile kernels,
    the tile kernels stay."""
    for precision, kernel in (("fp32", f32), ("fp64", f64)):
        b = lks.Batch(_designs(sizes, thermal), precision=precision, bind=False)
        assert b.launch_plan()[0] == kernel, precision
