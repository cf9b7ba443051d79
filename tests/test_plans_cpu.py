"""The rules that choose a kernel form, evaluated on the host (no GPU calls)."""
import pytest

import kct_inputs as ki
from tests.plan_util import BWD_BRICKS, BWD_DEEP, BWD_WAVES, plan_of


def plan(n, q, views, dtype="f32", projector="siddon"):
    """The forms of nx x ny x nz voxels of 120 / max mm with q detector pixels per voxel at the isocentre."""
    nx, ny, nz = n
    v = 120.0 / max(n)
    g = ki.ConeGeometry(nx, ny, nz, v, v, v, n_views=views, nu=int(1.45 * max(nx, ny) * q) + 3, nv=int(1.1 * nz * q) + 3,
                        du=2.0 * v / q, dv=2.0 * v / q, angle0=0.3)
    return plan_of(g, dtype, projector)


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


@pytest.mark.parametrize("projector, dtype", [("siddon", "f32"), ("siddon", "f64"), ("tt", "f32")])
@pytest.mark.parametrize("views", [1, 2, 3, 4, 5, 7, 9, 15, 16, 100])
def test_no_wavefront_waits_for_views_that_do_not_exist(views, projector, dtype):
    """Half as many view subsets would not do, and a single view has one."""
    for n in (12, 48, 96, 192, 256, 400):
        for q in (0.7, 1.25, 2.2, 6.0):
            p = plan((n, n, n), q, views, dtype, projector)
            if p["form"] == BWD_WAVES:
                assert p["sets"] == 1 or p["sets"] // 2 < views
                assert p["sets"] in (1, 2, 4, 8, 16)


def test_few_views_take_workgroup_bricks():
    assert plan((256, 256, 256), 1.25, 1)["form"] == BWD_BRICKS
    assert plan((192, 192, 192), 1.25, 2)["form"] == BWD_BRICKS
    assert plan((192, 192, 192), 1.25, 180)["form"] == BWD_WAVES
    assert plan((96, 96, 96), 1.25, 1)["form"] == BWD_WAVES
    assert plan((256, 256, 256), 1.25, 7)["form"] == BWD_BRICKS
    assert plan((256, 256, 256), 1.25, 8)["form"] == BWD_WAVES


@pytest.mark.parametrize("layers, tz", [(64, 32), (68, 16), (69, 32), (96, 32)])
def test_deepest_wave_bricks_are_mostly_filled(layers, tz):
    """They take all 32 layers: at least five sevenths of the last layers exist."""
    p = plan((256, 256, layers), 0.7, 60)
    assert (p["form"], p["tz"]) == (BWD_WAVES, tz)


def forward_tiles(nu, nv, views, rows, ws, in_place=0):
    import ctypes
    from paper_2110_13526_amd import _lib
    fn = _lib.load().kct_test_forward_tile
    out = (ctypes.c_int64 * 3)()
    for w in ws:
        fn(nu, nv, views, rows, in_place, ctypes.c_int64(w), out)
        yield tuple(out)


@pytest.mark.parametrize("in_place", [0, 1])
@pytest.mark.parametrize("nu, nv, views, rows", [(1, 1, 1, 1), (37, 65, 23, 1), (616, 480, 7, 4), (131, 129, 300, 2), (9, 200, 129, 3)])
def test_forward_tiles_cover_the_projection_once(nu, nv, views, rows, in_place):
    groups, bands = (nu + 3) // 4, (nv + 64 * rows - 1) // (64 * rows)
    tiles = set(forward_tiles(nu, nv, views, rows, range(groups * bands * views), in_place))
    assert len(tiles) == groups * bands * views
    assert all(0 <= c < groups and 0 <= k < views and 0 <= b < bands for c, k, b in tiles)


@pytest.mark.parametrize("in_place", [0, 1])
@pytest.mark.parametrize("nu, views", [(2**28 - 1, 1), (2**28 - 1, 7), (2**27, 15), (2**27 - 1, 2), (2**24, 127), (2**23 - 3, 250)])
def test_forward_tiles_of_the_widest_detectors(nu, views, in_place):
    """Detectors of one row whose column groups times a block of views pass 2^32."""
    groups = (nu + 3) // 4
    n = groups * views
    ws = [w for w in (0, 1, 2, groups - 1, groups, n // 2, n // 3, n - 2, n - 1) if w < n]
    tiles = list(forward_tiles(nu, 1, views, 1, ws, in_place))
    assert len(set(tiles)) == len(set(ws))
    assert all(0 <= c < groups and 0 <= k < views and b == 0 for c, k, b in tiles)


def test_detectors_beyond_the_column_offsets_are_refused():
    """32-byte column parameters are addressed by 32-bit offsets: 2^27 columns would wrap."""
    import ctypes
    import threading
    from paper_2110_13526_amd import _lib
    got = []

    def call():  # in a thread of its own: the message is the calling thread's
        vol = _lib.VolumeDesc(8, 8, 8, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0)
        out = (ctypes.c_int64 * 8)()
        cone = _lib.ConeDesc(1, 0.0, 6.28, None, 500.0, 1000.0, 2**27, 1, 1e-6, 1.0, 0.0, 0.0)
        got.append(_lib.load().kct_test_plan(ctypes.byref(vol), ctypes.byref(cone), 0, _lib.KCT_F32, out))
        got.append(_lib.load().kct_last_error())

    t = threading.Thread(target=call)
    t.start()
    t.join()
    assert got[0] == 1 and b"2^27 columns" in got[1]


def thin(nx, ny, nz, q, views=8):
    """A volume of at most 116 mm on a truncated 512 x 512 detector, q pixels per voxel."""
    v = 116.0 / max(nx, ny, nz)
    return ki.ConeGeometry(nx, ny, nz, v, v, v, n_views=views, nu=512, nv=512, du=2.0 * v / q, dv=2.0 * v / q, angle0=0.3)


@pytest.mark.parametrize("projector, dtype", [("siddon", "f32"), ("siddon", "f64"), ("tt", "f32")])
@pytest.mark.parametrize("n", [(1, 46340, 46340), (46340, 46340, 1), (1, 2**20, 2047), (2**20, 1, 2047), (2**20, 2047, 1),
                               (1, 2047, 2**20), (1290, 1290, 1290), (3, 26000, 26000), (1, 23170, 23170)])
def test_bricks_fit_one_launch(n, projector, dtype):
    """A grid has less than 2^32 threads."""
    for q in (0.7, 2.5, 3.2, 9.0):
        for views in (1, 2, 8):
            p = plan_of(thin(*n, q, views), dtype, projector)
            assert p["blocks"] * (64 * p["sets"] if p["form"] == BWD_WAVES else 256) < 2**32
            assert p["tz"] <= (16 if projector == "tt" else 32)
