"""Backprojection of volumes that fill only part of a brick's depth: the layers above the
volume's top are left out, in time and in the sums.

Tolerances against the FP64 oracle as for every form of the backprojection
(tests/test_gpu_forms.py, tests/test_gpu_tt_forms.py): relative L2 error 1e-5; per voxel 1e-4
(footprints 1e-3) of the largest value.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod

pytestmark = pytest.mark.gpu


def _geo(n, layers, q, views, **more):
    v = 120.0 / n
    du = 2.0 * v / q
    return ki.ConeGeometry(n, n, layers, v, v, v, n_views=views, nu=int(1.45 * n * q) + 3, nv=int(1.2 * layers * q) + 4,
                           du=du, dv=du, angle0=0.3, **more)


@pytest.mark.parametrize("projector", ["siddon", "tt"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("layers", [1, 3, 4, 5, 8, 9, 16, 17, 20, 31, 33, 37])
def test_partial_depth(layers, dtype, projector):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    tdt = {"f32": torch.float32, "f64": torch.float64}[dtype]
    back = {"siddon": oracle.backproject, "tt": oracle.tt_backproject}[projector]
    for n, q, views in ((41, 1.3, 5), (33, 2.6, 3), (49, 0.7, 9)):
        g = _geo(n, layers, q, views, cz=0.7, off_v=-0.4)
        G = geometry(g)
        G.set_projector(projector)
        say(f"[thin] {projector} {dtype} vol {g.vol_shape} proj {g.proj_shape}")
        y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 3)).to(dev()).to(tdt)
        r, ref = to_np(kct.backproject(G, y)), back(g, to_np(y))
        worst = float(np.abs(r - ref).max() / ref.max())
        assert rel(r, ref) < 1e-5
        assert worst < (1e-4 if projector == "siddon" else 1e-3)


def test_one_layer_costs_less_than_a_full_brick():
    """One layer takes at most 0.7 of the time of sixteen with the same detector (a
    quarter of the voxels are summed, beside the staging of a smaller shadow)."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    times = []
    v = 120.0 / 1024
    for layers in (1, 16):
        G = geometry(ki.ConeGeometry(1024, 1024, layers, v, v, v, n_views=60, nu=1039, nv=17, du=2.0 * v / 0.7,
                                     dv=2.0 * v / 0.7, angle0=0.3))
        y = torch.ones(G.proj_shape, device=dev())
        out = torch.empty(G.vol_shape, device=dev())
        events = [torch.cuda.Event(enable_timing=True) for _ in range(11)]
        kct.backproject(G, y, out=out)
        for e in events:
            e.record()
            kct.backproject(G, y, out=out)
        torch.cuda.synchronize()
        times.append(min(a.elapsed_time(b) for a, b in zip(events, events[1:])))
    say(f"[thin] 1 layer {times[0]:.3f} ms, 16 layers {times[1]:.3f} ms")
    assert times[0] < 0.7 * times[1]
