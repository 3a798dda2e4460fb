"""bench.py names the kernels that run, and a shape it reports can be given back
to it (planning only, no GPU)."""
import glob
import os
import re

import pytest

import bench
from paper_2411_03090_amd import lks, workloads as W

SOURCES = {os.path.basename(f): open(f).read() for f in glob.glob(os.path.join(bench.CSRC, "*"))}


def _steady(nx, ny, precision):
    return lks.LKS(W.steady_channel_uniform(nx, ny, n_fwd=4, n_adj=4), precision=precision,
                   bind=False)


def test_counters_are_tied_to_every_kernel_source():
    kernels = {f for f, s in SOURCES.items() if "__global__" in s or "__device__" in s}
    assert kernels - set(bench.KERNEL_SOURCES) <= {"lks_runtime.hip"}  # (a flag's reset)


@pytest.mark.parametrize("nx,precision,dtype,fwd,adj", [
    (512, "fp64", "double", ("lks_multi_kernel<double, false>", 3),
     ("alks_multi_kernel<double, false>", 2)),
    (2048, "fp32", "float", ("lks_march_kernel<float, 2>", 2), ("alks_march_kernel<float, 2>", 2)),
    (1024, "fp32", "float", ("lks_step_kernel<float, false, {ty}>", 1),
     ("alks_step_kernel<float, false, {ty}>", 1))])
def test_names_are_those_of_the_kernels_that_run(nx, precision, dtype, fwd, adj):
    c = _steady(nx, nx, precision)
    for sweep, (name, steps) in (("fwd", fwd), ("adj", adj)):
        want = name.replace("{ty}", str(c.launch_shape()[0])), steps
        assert bench.sweep_kernel(c, sweep, dtype, False) == want
    c.set_tile_rows(4)
    c.set_steps_per_launch(2, 1)
    assert bench.sweep_kernel(c, "fwd", dtype, False) == (f"lks_step2_kernel<{dtype}, false, 4>", 2)


@pytest.mark.parametrize("many", ["", "batch", "ubatch"])
@pytest.mark.parametrize("kernel", lks.KERNELS)
def test_every_named_kernel_exists(kernel, many):
    if (kernel, many) == ("march", "ubatch"):
        return  # unsteady batches do not march
    for sweep in ("fwd", "adj"):
        name = bench.kernel_name(sweep, "float", False, kernel, 1, 4, many).split("<")[0]
        assert any(re.search(rf"__global__[^;{{]*\b{name}\(", s) for s in SOURCES.values()), name


@pytest.mark.parametrize("nx,precision", [(64, "fp64"), (512, "mixed"), (2048, "fp32")])
def test_reported_shapes_can_be_given_back(nx, precision):
    a, b, old = (_steady(nx, nx, precision) for _ in range(3))
    bench.apply_shape(b, list(bench.shape_dict(a).values()))
    assert b.launch_plan() == a.launch_plan()
    assert bench.shape_dict(b) == bench.shape_dict(a)
    bench.apply_shape(old, [8, 1, 1])  # a line without the kernels
    assert old.launch_plan() == (("tile", 1), ("tile", 1))
    wls = [W.steady_channel_uniform(64, 64, seed=d, n_fwd=4, n_adj=4) for d in range(3)]
    b = lks.Batch(wls, precision="fp32", bind=False)
    shape = bench.batch_shape_dict(b, 8)
    b.set_tile_rows(8)
    assert bench.batch_shape_dict(b, 8)["forward_kernel"] == "tile"
    bench.apply_batch_shape(b, list(shape.values()))
    assert bench.batch_shape_dict(b, 8) == shape


def test_roofline_of_several_steps_counts_one_pass_too():
    r = bench.roofline("nowhere", "k", ("2d", "fwd"), "float", 3000, 10.0, 3)
    assert r["achieved"] == pytest.approx(28 * 3000 / 10e-6 / 1e9)
    assert r["one_pass_achieved"] == pytest.approx(28 * 1000 / 10e-6 / 1e9)
    assert r["steps_per_launch"] == 3
    assert "one_pass_achieved" not in bench.roofline("nowhere", "k", ("2d", "fwd"), "float", 9, 1.0)
