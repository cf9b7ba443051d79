"""16-bit storage in the backprojection's wave forms 4, 8 and 32 voxels deep, and the
squared weights of the footprint pair's 4- and 8-deep forms, against the FP64 oracle of
the stored values.

Tolerances: the single-precision sum as in tests/test_gpu_forms.py and
tests/test_gpu_tt_forms.py (per voxel 1e-4, footprints 1e-3, of the largest value), then one
rounding to the storage type (8 or 11 significant bits); squared weights twice the
error of a weight.
"""
import numpy as np
import pytest

import kct_inputs as ki
import oracle
from tests.gpu_util import dev, geometry, rel, say, to_np, torch_mod
from tests.plan_util import BWD_WAVES, plan_of
from tests.test_gpu_forms import FORMS
from tests.test_gpu_tt_forms import FORMS as TT_FORMS

pytestmark = pytest.mark.gpu

DEPTHS = {
    "siddon": {"4x16": 4, "4x8_columns_chunked": 4, "4x16_rows_chunked": 4, "8x16": 8, "8x8": 8, "32x4": 32},
    "tt": {"rows_65": 4, "depth_4_columns_chunked": 4, "depth_8": 8},
}
CASES = [(p, n) for p in sorted(DEPTHS) for n in sorted(DEPTHS[p])]


@pytest.mark.parametrize("dtype, bits", [("bf16", 8), ("f16", 11)])
@pytest.mark.parametrize("projector, name", CASES)
def test_16_bit_storage(projector, name, dtype, bits):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    g = (FORMS if projector == "siddon" else TT_FORMS)[name]
    p = plan_of(g, dtype, projector)
    assert (p["form"], p["tz"]) == (BWD_WAVES, DEPTHS[projector][name])
    G = geometry(g)
    G.set_projector(projector)
    say(f"[storage forms] {projector} {name} {dtype}: vol {g.vol_shape} proj {g.proj_shape}")
    y = torch.from_numpy(1.0 + 0.5 * ki.random_projections(g, 3)).to(dev()).to({"bf16": torch.bfloat16, "f16": torch.float16}[dtype])
    r = to_np(kct.backproject(G, y).double())
    ref = (oracle.backproject if projector == "siddon" else oracle.tt_backproject)(g, to_np(y.double()))
    single = (1e-4 if projector == "siddon" else 1e-3) * ref.max()
    assert np.all(np.abs(r - ref) <= single + 2.0 ** -bits * (np.abs(ref) + single) + 2.0 ** -24)


@pytest.mark.parametrize("name", sorted(DEPTHS["tt"]))
def test_tt_diag_normal(name):
    import paper_2110_13526_amd as kct
    g = TT_FORMS[name]
    assert plan_of(g, "f32", "tt")["tz"] == DEPTHS["tt"][name]
    G = geometry(g)
    G.set_projector("tt")
    d, ref = to_np(kct.diag_normal(G)), oracle.tt_diag_normal(g)
    say(f"[storage forms] tt diag {name}: rel {rel(d, ref):.2e}, largest {np.abs(d - ref).max() / ref.max():.2e}")
    assert rel(d, ref) < 2e-5
    assert np.abs(d - ref).max() < 2e-3 * ref.max()
