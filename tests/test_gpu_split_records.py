"""The backprojection with its staged records split into row factors and per-ray
values: bricks 4, 8 and 16 voxels deep with four view subsets, chunks of more rows
than a staged row table holds, and a detector row parallel to the z-planes, against the
FP64 oracle; and the workgroup bricks against the double-precision accumulation of the
same single-precision weights, whose records are whole.

Tolerances against the oracle as for every form of the backprojection
(tests/test_gpu_forms.py): relative L2 error 1e-5, per voxel 1e-4 of the largest value.
Against double accumulation, per voxel 3e-6 of its own value: at most 2 views x 18
non-negative terms, each rounded once or twice to 2^-24 relative.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod
from tests.test_gpu_forms import _cube

pytestmark = pytest.mark.gpu

# name -> geometry: depth and subsets that the rule takes for it
SPLIT = {
    "4x4": _cube(145, 137, 101, 3.2, 5),
    "8x4": _cube(177, 169, 150, 2.0, 5),
    "16x4": _cube(177, 169, 281, 1.2, 5),
    "4x16_rows_chunked": _cube(9, 9, 6, 22.0, 18),
    "parallel_row": ki.ConeGeometry(33, 33, 31, 3.0, 3.0, 3.0, n_views=9, nu=71, nv=41, du=4.0, dv=4.0),
}


@pytest.mark.parametrize("name", sorted(SPLIT))
def test_split_records(name):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = SPLIT[name]
    say(f"[split] {name}: vol {g.vol_shape} proj {g.proj_shape}")
    y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 5)).to(dev()).to(torch.float32)
    r = to_np(kct.backproject(geometry(g), y))
    ref = oracle.backproject(g, to_np(y))
    assert rel(r, ref) < 1e-5
    assert np.abs(r - ref).max() < 1e-4 * ref.max()


def test_split_bricks_weights():
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = _cube(385, 371, 345, 1.2, 2, nv_share=0.9)
    G = geometry(g)
    y = torch.from_numpy(1.0 + 0.5 * np.abs(ki.random_projections(g, 5))).to(dev()).to(torch.float32)
    r = kct.backproject(G, y).to(torch.float64)
    ref = kct.backproject(G, y.to(torch.float64))
    assert float(ref.max()) > 0.0
    assert bool(((r - ref).abs() <= 3e-6 * ref.abs()).all())
