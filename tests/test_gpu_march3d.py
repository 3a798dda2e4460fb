"""The D3Q19 z-marches at the sizes where their tiling changes: fewer columns
than a tile, a second tile that overlaps the first, the fewest planes (the
periodic axis of three planes, whose halo wraps more than once), and several
chunks of the z axis.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_3d as base  # noqa: E402
from paper_2411_03090_amd import workloads as W  # noqa: E402


def _box(nx, ny, nz):
    wl = W.periodic_box3(nx, ny, nz, nu=0.08, thermal=True, Pr=6.0)
    wl.alpha_max, wl.Ks_over_Kf = 0.7, 3.0
    wl.gamma = np.random.default_rng(2).uniform(0.05, 1.0, (nz, ny, nx))
    wl.mask = wl.mask.copy()
    wl.mask[1, 2:4, 3] |= W.TAG_PROBE
    wl.objective = W.OBJ_HEAT
    return wl


SIZES = {
    "box_5x4x3": lambda: _box(5, 4, 3),
    "box_66x5x4": lambda: _box(66, 5, 4),
    "duct_65x9x5": lambda: base._duct(65, 9, 5),
    "duct_12x6x41": lambda: base._duct(12, 6, 41),
    "duct_8x8x7": lambda: base._duct(8, 8, 7),  # one plane of packed x-face moments
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(SIZES))
def test_marches_at_tile_edges(case, prec, monkeypatch):
    """One LKS and one ALKS step match the oracle, and the fused ALKS step the
    three passes."""
    monkeypatch.setitem(base.CASES, case, SIZES[case])
    base.test_single_forward_step_3d(case, prec)
    base.test_single_adjoint_step_3d(case, prec)
    base.test_fused_adjoint_equals_three_passes(case, prec)
