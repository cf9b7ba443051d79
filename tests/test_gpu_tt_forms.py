"""The TT footprint pair's forms in single precision, against the FP64 oracle: one and
two detector rows per lane with partial bands and column groups, backprojection
bricks 4, 8 and 16 voxels deep with the views in 4, 8 or 16 subsets, shadows of
several staged chunks, and thin layers far from the source plane, where the images
of neighbouring z-planes overlap.

Tolerances: relative L2 error 1e-5, the bound of every single-precision projection;
per value 1e-3 of the largest: a footprint's breakpoints carry half a unit of a
detector coordinate below 512 (3e-5 pixel), a weight is the difference of four of
them, and all weights of a value may err alike.  A dropped voxel column, z-cell or
pixel would cost its value about 1 / (terms of the sum), above 1e-2 for all but
slivers.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_dev, to_np, torch_mod

pytestmark = pytest.mark.gpu


def _geo(n, q, views, nu=None, nv=None, vz=1.0, **more):
    nx, ny, nz = n
    v = 100.0 / max(nx, ny)
    du = 2.0 * v / q
    nu = nu or int(1.4 * max(nx, ny) * q) + 3
    nv = nv or int(1.1 * nz * vz * q) + 3
    return ki.ConeGeometry(nx, ny, nz, v, v, v * vz, n_views=views, nu=nu, nv=nv, du=du, dv=du, angle0=0.3, **more)


FORMS = {
    "one_column": _geo((9, 8, 7), 1.0, 3, nu=1, nv=1),
    "rows_64": _geo((33, 29, 40), 1.3, 5, nv=64, cx=1.2, cy=-0.7, cz=2.1, off_u=0.9, off_v=-1.4),
    "rows_65": _geo((33, 29, 40), 1.3, 5, nu=9, nv=65),
    "rows_129": _geo((21, 50, 90), 1.3, 4, nv=129),
    "depth_16": _geo((49, 41, 65), 0.8, 17),
    "depth_16_sets_8": _geo((97, 97, 101), 0.7, 9),
    "depth_16_sets_4": _geo((130, 130, 125), 0.7, 6),
    "depth_8": _geo((49, 41, 51), 2.4, 18),
    "depth_4_columns_chunked": _geo((41, 33, 24), 6.0, 9),
    "depth_4_rows_chunked": _geo((9, 9, 6), 26.0, 5),
    "overlap": _geo((25, 21, 90), 1.1, 7, nv=80, vz=0.125, cz=60.0, off_v=120.0),
}


@pytest.mark.parametrize("name", sorted(FORMS))
def test_tt_forms(name):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = FORMS[name]
    G = geometry(g)
    G.set_projector("tt")
    say(f"[tt forms] {name}: vol {g.vol_shape} proj {g.proj_shape}")
    x = (1.0 + 0.5 * ki.random_volume(g, 1)).astype(np.float32)
    bs = [kct.project(G, to_dev(x), transposed_copy=copy) for copy in (True, False)]
    assert torch.equal(*bs)
    b, ref = to_np(bs[0]), oracle.tt_project(g, x.astype(np.float64))
    assert rel(b, ref) < 1e-5
    assert np.abs(b - ref).max() < 1e-3 * ref.max()
    y = (1.0 + 0.5 * ki.random_projections(g, 2)).astype(np.float32)
    r, ref = to_np(kct.backproject(G, to_dev(y))), oracle.tt_backproject(g, y.astype(np.float64))
    assert rel(r, ref) < 1e-5
    assert np.abs(r - ref).max() < 1e-3 * ref.max()


def test_tt_overlap_weights_bitwise_identical():
    """Sorted breakpoints (overlapping planes): the pair holds the same weight bits."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = FORMS["overlap"]
    G = geometry(g)
    G.set_projector("tt")
    checked = 0
    for j in np.random.default_rng(12).choice(g.n_vox, 6, replace=False):
        x = torch.zeros(g.n_vox, device=dev())
        x[j] = 1.0
        col = kct.project(G, x.view(g.vol_shape)).view(-1)
        for i in torch.nonzero(col).view(-1).cpu().numpy()[:8]:
            y = torch.zeros(g.n_rays, device=dev())
            y[i] = 1.0
            row = kct.backproject(G, y.view(g.proj_shape)).view(-1)
            assert row[j].view(torch.int32).item() == col[i].view(torch.int32).item()
            checked += 1
    assert checked > 0
