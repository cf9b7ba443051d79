"""Backprojections of one to seven views, whose subsets are fewer than the groups that
partial sums are added in, against the FP64 oracle.

Tolerances as for every form of the backprojection (tests/test_gpu_forms.py,
tests/test_gpu_tt_forms.py): relative L2 error 1e-5; per voxel 1e-4 (footprints 1e-3) of the
largest value, and twice the relative error for squared weights.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod
from tests.plan_util import BWD_BRICKS, BWD_WAVES, plan_of
from tests.test_gpu_forms import _cube

pytestmark = pytest.mark.gpu

SIZES = [(49, 41, 51, 1.7), (33, 37, 29, 1.0), (97, 97, 61, 1.2), (21, 25, 18, 5.0)]


@pytest.mark.parametrize("projector, dtype", [("siddon", "f32"), ("siddon", "f64"), ("tt", "f32")])
@pytest.mark.parametrize("views", [1, 2, 3, 5, 7])
def test_few_views(views, projector, dtype):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    back = {"siddon": oracle.backproject, "tt": oracle.tt_backproject}[projector]
    for nx, ny, nz, q in SIZES:
        g = _cube(nx, ny, nz, q, views)
        G = geometry(g)
        G.set_projector(projector)
        p = plan_of(g, dtype, projector)
        say(f"[few views] {projector} {dtype} vol {g.vol_shape} proj {g.proj_shape} form {p['form']} {p['tz']} x {p['sets']}")
        y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 3)).to(dev()).to(tdt)
        r, ref = to_np(kct.backproject(G, y)), back(g, to_np(y))
        worst = float(np.abs(r - ref).max() / ref.max())
        assert rel(r, ref) < 1e-5
        assert worst < (1e-4 if projector == "siddon" else 1e-3)


def test_one_view_bricks():
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = _cube(129, 113, 101, 1.25, 1)
    assert plan_of(g)["form"] == BWD_BRICKS and plan_of(_cube(129, 113, 101, 1.25, 9))["form"] == BWD_WAVES
    y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 3)).to(dev()).to(torch.float32)
    r, ref = to_np(kct.backproject(geometry(g), y)), oracle.backproject(g, to_np(y))
    assert rel(r, ref) < 1e-5
    assert np.abs(r - ref).max() < 1e-4 * ref.max()


def test_diag_normal_of_one_and_two_views():
    import paper_2110_13526_amd as kct
    for views in (1, 2):
        for nx, ny, nz, q in SIZES[:3]:
            g = _cube(nx, ny, nz, q, views)
            assert rel(to_np(kct.diag_normal(geometry(g))), oracle.diag_normal(g)) < 2e-5
