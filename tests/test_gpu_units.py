"""The unit of length does not matter: lengths scaled by a power of two scale every
weight of the backprojection, and so every result, by it exactly, rows parallel to
the z-planes included."""
import dataclasses

import pytest

import kct_inputs as ki
from tests.gpu_util import dev, geometry, say, torch_mod
from tests.plan_util import BWD_BRICKS, BWD_DEEP, BWD_WAVES, plan_of
from tests.test_gpu_forms import _cube

pytestmark = pytest.mark.gpu

LENGTHS = ("vx", "vy", "vz", "du", "dv", "sid", "sdd", "cx", "cy", "cz", "off_u", "off_v")


def _odd(g):
    return dataclasses.replace(g, nv=g.nv | 1)


FORMS = {
    "split_records": (_odd(_cube(33, 37, 29, 1.2, 9)), BWD_WAVES),
    "whole_records": (_odd(_cube(121, 115, 97, 0.6, 8)), BWD_WAVES),
    "bricks": (_odd(_cube(129, 113, 101, 1.25, 1)), BWD_BRICKS),
    "deep_bricks": (_odd(_cube(256, 256, 256, 0.7, 1)), BWD_DEEP),
}


@pytest.mark.parametrize("power", [-40, -13, 20, 40])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_units(name, dtype, power):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g, form = FORMS[name]
    scaled = dataclasses.replace(g, **{f: getattr(g, f) * 2.0**power for f in LENGTHS})
    if dtype == "f32":
        assert plan_of(g)["form"] == plan_of(scaled)["form"] == form
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    y = torch.from_numpy(ki.random_projections(g, 5)).to(dev()).to(tdt)
    r, s = kct.backproject(geometry(g), y), kct.backproject(geometry(scaled), y)
    say(f"[units] {name} {dtype} 2^{power}: largest {float(r.abs().max())} {float(s.abs().max())}")
    assert bool(torch.isfinite(r).all()) and float(r.abs().max()) > 0.0
    assert torch.equal(s, r * 2.0**power)
