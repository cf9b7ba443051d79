"""A flat volume of 5.4e8 voxels, whose bricks of 1 x 8 x 4 voxels times four view subsets
are more threads than a launch can have: <A^T y, x> = <y, A x> for an x in a small
region.  Tolerance 1e-5, the bound of every single-precision projection."""
import pytest

from tests.gpu_util import dev, geometry, say, torch_mod
from tests.test_plans_cpu import thin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("projector", ["siddon", "tt"])
def test_flat_volume(projector):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = thin(1, 23300, 23300, 3.2, views=8)
    G = geometry(g)
    G.set_projector(projector)
    say(f"[flat] {projector} vol {g.vol_shape} proj {g.proj_shape}")
    gen = torch.Generator(device=dev())
    gen.manual_seed(1)
    y = torch.rand(g.proj_shape, generator=gen, device=dev())
    r = kct.backproject(G, y)
    x = torch.zeros(g.vol_shape, device=dev())
    part = (slice(11600, 11700), slice(11610, 11690), slice(None))
    x[part] = torch.rand(x[part].shape, generator=gen, device=dev())
    left = float((r[part].double() * x[part].double()).sum())
    b = kct.project(G, x)
    right = float((b.double() * y.double()).sum())
    say(f"[flat] {left!r} {right!r}")
    assert right > 0.0 and abs(left - right) < 1e-5 * right
