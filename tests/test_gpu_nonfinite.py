"""A detector value that is not finite reaches the voxel columns that its detector column
hits and no others (footprints: the voxels whose footprint meets its pixel and no
others), in every form of the backprojection; all other voxels keep their value."""
import pytest

import kct_inputs as ki
from tests.gpu_util import dev, geometry, say, torch_mod
from tests.plan_util import BWD_BRICKS, BWD_DEEP, BWD_WAVES, plan_of
from tests.test_gpu_forms import _cube

pytestmark = pytest.mark.gpu

FORMS = {
    "4": (_cube(41, 37, 29, 3.3, 12), BWD_WAVES, 4),
    "8": (_cube(65, 65, 71, 1.9, 9), BWD_WAVES, 8),
    "16": (_cube(97, 97, 101, 1.2, 9), BWD_WAVES, 16),
    "32": (_cube(125, 123, 121, 0.7, 9), BWD_WAVES, 32),
    "bricks": (_cube(193, 193, 113, 1.25, 3), BWD_BRICKS, 16),
    "deep_bricks": (_cube(256, 256, 256, 0.7, 4), BWD_DEEP, 32),
}


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_value_stays_in_the_columns_it_hits(name, dtype, value):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g, form, tz = FORMS[name]
    if dtype == "f32":
        p = plan_of(g)
        assert (p["form"], p["tz"]) == (form, tz)
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    G = geometry(g)
    y = torch.rand(g.proj_shape, device=dev()).to(tdt)
    clean = kct.backproject(G, y)
    for k in range(min(3, g.n_views)):
        for u in (g.nu // 2, g.nu // 2 - 3, g.nu // 4, (3 * g.nu) // 4, g.nu // 5):
            v = g.nv // 2 + 2
            column = torch.zeros_like(y)
            column[k, :, u] = 1.0
            hit = (kct.backproject(G, column) != 0).any(dim=0)  # voxel columns that detector column u hits
            one = torch.zeros_like(y)
            one[k, v, u] = 1.0
            ray = kct.backproject(G, one) != 0
            bad = y.clone()
            bad[k, v, u] = value
            r = kct.backproject(G, bad)
            spread = ~torch.isfinite(r)
            assert bool((spread | ~ray).all())
            assert not bool((spread & ~hit[None]).any()), (k, u, int((spread & ~hit[None]).sum()), int(spread.sum()))
            assert torch.equal(r[~spread], clean[~spread])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("q", [1.0, 2.0, 4.0])
def test_footprints_only_touched(q, value):
    """Voxels whose footprint ends exactly on the pixel's edge, in a view along an axis."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    n, v = 16, 2.0
    g = ki.ConeGeometry(n, n, n, v, v, v, n_views=1, nu=64, nv=64, du=2.0 * v / q, dv=2.0 * v / q, angle0=0.0)
    G = geometry(g)
    G.set_projector("tt")
    y = torch.rand(g.proj_shape, device=dev())
    for u, w in ((31, 31), (32, 32), (32, 40), (25, 31)):
        one = torch.zeros_like(y)
        one[0, w, u] = 1.0
        met = kct.backproject(G, one) != 0
        bad = y.clone()
        bad[0, w, u] = value
        spread = ~torch.isfinite(kct.backproject(G, bad))
        say(f"[footprints] q {q} pixel {(u, w)}: met {int(met.sum())}, spread {int(spread.sum())}")
        assert torch.equal(spread, met)
