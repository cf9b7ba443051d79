"""The kernel forms that the library's rules take for a geometry (host arithmetic, no GPU calls)."""
import ctypes

BWD_WAVES, BWD_BRICKS, BWD_DEEP = 0, 1, 2
KEYS = ("rows", "divided", "in_place", "fwd_blocks", "form", "tz", "sets", "blocks")


def plan_of(g, dtype="f32", projector="siddon"):
    """g: a geometry description (kct_inputs.ConeGeometry or any object with its fields)."""
    from paper_2110_13526_amd import _lib
    vol = _lib.VolumeDesc(g.nx, g.ny, g.nz, g.vx, g.vy, g.vz, g.cx, g.cy, g.cz)
    cone = _lib.ConeDesc(g.n_views, g.angle0, g.arc, None, g.sid, g.sdd, g.nu, g.nv, g.du, g.dv, g.off_u, g.off_v)
    out = (ctypes.c_int64 * len(KEYS))()
    code = {"f32": _lib.KCT_F32, "bf16": _lib.KCT_BF16, "f16": _lib.KCT_F16, "f64": _lib.KCT_F64}[dtype]
    proj = {"siddon": _lib.PROJECTOR_SIDDON, "tt": _lib.PROJECTOR_TT}[projector]
    assert _lib.load().kct_test_plan(ctypes.byref(vol), ctypes.byref(cone), proj, code, out) == 0
    return dict(zip(KEYS, out))
