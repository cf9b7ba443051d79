"""The forms of the backprojection: by wavefronts with bricks 4, 8, 16 and 32
voxels deep and the views in 4, 8 or 16 subsets, against the FP64 oracle at
sizes with partial bricks, one subset longer than another, and shadows that take
several staged chunks in either direction; and the batched form's sums against
the separate solves'.

Tolerances: relative L2 error 1e-5, the bound of every single-precision
backprojection; per voxel 1e-4 of the largest value: a crossing is resolved to
about 1e-5 of a voxel, a weight is the difference of two, and all of a voxel's
weights (their sum at most the largest value) may err alike.  A candidate ray
that the bounds dropped would cost its voxel about 1 / (views x rays per view),
above 1e-3 here.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod

pytestmark = pytest.mark.gpu


def _cube(nx, ny, nz, q, views, nv_share=1.1, **more):
    """nx x ny x nz voxels of 120 / max mm, q detector pixels per voxel at the isocentre."""
    v = 120.0 / max(nx, ny, nz)
    du = 2.0 * v / q
    n = max(nx, ny)
    return ki.ConeGeometry(nx, ny, nz, v, v, v, n_views=views, nu=int(1.45 * n * q) + 3, nv=int(nv_share * nz * q) + 3,
                           du=du, dv=du, angle0=0.3, **more)


# name -> geometry: depth and subsets that the rule takes for it
FORMS = {
    "4x16": _cube(17, 9, 5, 2.0, 21),
    "4x16_fewer_views": _cube(17, 9, 5, 2.0, 5),
    "4x8_columns_chunked": _cube(57, 41, 63, 4.5, 9, nv_share=0.4),
    "4x16_rows_chunked": _cube(9, 9, 6, 14.0, 18),
    "8x16": _cube(49, 41, 51, 1.7, 33, cx=2.1, cy=-1.3, cz=0.7, off_u=0.3, off_v=-0.4),
    "8x8": _cube(65, 65, 71, 1.7, 9),
    "8x4": _cube(137, 129, 60, 1.7, 6),
    "16x16": _cube(49, 41, 65, 1.0, 17),
    "16x8": _cube(97, 97, 101, 1.2, 9),
    "16x4": _cube(130, 130, 125, 1.2, 6),
    "32x4": _cube(125, 123, 121, 0.7, 6),
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_backprojection_forms(name, dtype):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = FORMS[name]
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    say(f"[forms] {name} {dtype}: vol {g.vol_shape} proj {g.proj_shape}")
    y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 3)).to(dev()).to(tdt)
    r = to_np(kct.backproject(geometry(g), y))
    ref = oracle.backproject(g, to_np(y))
    assert rel(r, ref) < 1e-5
    assert np.abs(r - ref).max() < 1e-4 * ref.max()


def test_forms_diag_normal():
    """Squared weights through the same forms: per voxel twice the relative error of a weight."""
    import paper_2110_13526_amd as kct
    for name in ("4x16_rows_chunked", "8x16", "16x16"):
        g = FORMS[name]
        d = to_np(kct.diag_normal(geometry(g)))
        ref = oracle.diag_normal(g)
        assert rel(d, ref) < 2e-5, name


def test_batch_sums_equal_separate_solves():
    """Four wavefronts take the subsets of the separate solve in turns: the same bits."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    names = ["4x16", "4x8_columns_chunked", "8x16", "8x8", "16x16", "16x8", "32x4"]
    geoms = [geometry(FORMS[n]) for n in names]
    gen = torch.Generator(device=dev())
    gen.manual_seed(9)
    bs = [torch.rand(g.proj_shape, generator=gen, device=dev()) for g in geoms]
    batch = kct.Batch(geoms)
    xs, infos = batch.cgls(bs, 2)
    for n, g, b, x, i in zip(names, geoms, bs, xs, infos):
        x1, i1 = kct.cgls(g, b, 2)
        assert torch.equal(x, x1), n
        assert i.nb == i1.nb, n
    batch.close()
