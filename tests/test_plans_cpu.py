"""The rules that choose a kernel form, evaluated on the host (no GPU calls)."""
import ctypes
import math

import pytest

F32, F64 = 0, 3
SIDDON, TT = 0, 1
BWD_WAVES, BWD_BRICKS, BWD_DEEP = 0, 1, 2


def plan(n, q, views, dtype="f32", projector="siddon", detector=None):
    """The forms of nx x ny x nz voxels of 120 / max mm with q detector pixels per voxel at the isocentre."""
    from paper_2110_13526_amd import _lib
    L = _lib.load()
    nx, ny, nz = n
    v = 120.0 / max(n)
    nu, nv = detector or (int(1.45 * max(nx, ny) * q) + 3, int(1.1 * nz * q) + 3)
    vol = _lib.VolumeDesc(nx, ny, nz, v, v, v, 0.0, 0.0, 0.0)
    cone = _lib.ConeDesc(views, 0.3, 2.0 * math.pi, None, 500.0, 1000.0, nu, nv, 2.0 * v / q, 2.0 * v / q, 0.0, 0.0)
    out = (ctypes.c_int64 * 8)()
    code = {"f32": _lib.KCT_F32, "f64": _lib.KCT_F64}[dtype]
    proj = {"siddon": _lib.PROJECTOR_SIDDON, "tt": _lib.PROJECTOR_TT}[projector]
    assert L.kct_test_plan(ctypes.byref(vol), ctypes.byref(cone), proj, code, out) == 0
    keys = ("rows", "divided", "in_place", "fwd_blocks", "form", "tz", "sets", "blocks")
    return dict(zip(keys, out))


@pytest.mark.parametrize("projector, dtype", [("siddon", "f32"), ("siddon", "f64"), ("tt", "f32")])
@pytest.mark.parametrize("q", [0.7, 1.25, 2.2, 6.0])
@pytest.mark.parametrize("layers", [1, 2, 4, 5, 8, 9, 16])
def test_bricks_no_deeper_than_the_volume(layers, q, projector, dtype):
    """A wave-form brick of half the depth would not hold all layers."""
    for n in (9, 64, 300):
        p = plan((n, n, layers), q, 12, dtype, projector)
        if p["form"] == BWD_WAVES:
            assert p["tz"] == 4 or p["tz"] // 2 < layers


def test_double_precision_has_no_deep_bricks_for_thin_volumes():
    for layers in (1, 8, 20, 40):
        assert plan((1024, 1024, layers), 0.7, 12, "f64")["form"] != BWD_DEEP
    assert plan((512, 512, 256), 0.7, 12, "f64")["form"] == BWD_DEEP
