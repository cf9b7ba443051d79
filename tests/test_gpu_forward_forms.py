"""The forms of the forward projection: one to four detector rows per lane, and
walks divided among four wavefronts, against the FP64 oracle at detectors with
partial bands, few columns and few views, and the batched form's sums against
the separate solves'.

Tolerances: relative L2 error 1e-5, the bound of every single-precision
projection; per ray 1e-4 of the largest value (a crossing is resolved to about
1e-5 of a voxel, a weight is the difference of two, and all weights of a ray may
err alike).  A piece of a walk that was left out or taken twice would change its ray
by about 1 / (cells along the ray), above 5e-3 here.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod

pytestmark = pytest.mark.gpu


def _geo(n, nu, nv, views, **more):
    nx, ny, nz = n
    v = 120.0 / max(n)
    return ki.ConeGeometry(nx, ny, nz, v, v, v, n_views=views, nu=nu, nv=nv, du=330.0 / nu, dv=280.0 / nv, angle0=0.3, **more)


# rows per lane that the rule takes, d: divided
FORMS = {
    "1d_one_column": _geo((17, 13, 9), 1, 7, 5),
    "1d": _geo((33, 29, 21), 37, 64, 11, cx=1.2, cy=-0.7, cz=2.1, off_u=0.9, off_v=-1.4),
    "1": _geo((40, 47, 30), 133, 61, 41),
    "2d": _geo((33, 29, 40), 37, 65, 23),
    "2": _geo((40, 47, 30), 133, 128, 41),
    "3": _geo((61, 50, 40), 67, 190, 9),
    "3_two_bands": _geo((61, 50, 40), 35, 380, 9),
    "4": _geo((61, 50, 40), 67, 200, 9),
    "4_two_bands": _geo((50, 61, 40), 35, 511, 130),
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_forward_forms(name, dtype):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = FORMS[name]
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    say(f"[forward forms] {name} {dtype}: vol {g.vol_shape} proj {g.proj_shape}")
    x = torch.from_numpy(1.0 + 0.5 * ki.random_volume(g, 3)).to(dev()).to(tdt)
    ref = oracle.project(g, to_np(x))
    bs = [kct.project(geometry(g), x, transposed_copy=copy) for copy in (True, False)]
    assert torch.equal(*bs)
    b = to_np(bs[0])
    assert rel(b, ref) < 1e-5
    assert np.abs(b - ref).max() < 1e-4 * ref.max()


def test_batch_sums_equal_separate_solves():
    """Divided walks are taken share by share in a batch: the same bits."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    names = ["1d", "1", "2d", "2", "3", "4_two_bands"]
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
