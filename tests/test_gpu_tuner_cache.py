"""The batched form's tuner keeps its choices by what they depend on: voxels of another
width in pixels are another choice, and choices of an older file format are not taken."""
import pytest

import kct_inputs as ki

from tests.gpu_util import dev, geometry, rel, to_np, torch_mod
from tests.test_gpu_forms import _cube

pytestmark = pytest.mark.gpu


def _lines(path):
    return [ln.split() for ln in open(path).read().splitlines() if ln.strip()]


def test_equal_counts_of_another_magnification(tmp_path):
    import paper_2110_13526_amd as kct
    a = _cube(48, 48, 48, 1.0, 9)
    b = type(a)(**{**{f: getattr(a, f) for f in kct.Geometry.FIELDS}, "du": a.du / 2, "dv": a.dv / 2})
    assert a.proj_shape == b.proj_shape
    cache = str(tmp_path / "tune.txt")
    batch = kct.Batch([geometry(a), geometry(b), geometry(a)])
    batch.tune(cache=cache)
    batch.close()
    assert len({ln[0] for ln in _lines(cache)}) == len(_lines(cache)) == 2


def test_older_lines_are_not_taken(tmp_path):
    import paper_2110_13526_amd as kct
    g = _cube(48, 48, 48, 1.0, 9)
    cache = str(tmp_path / "tune.txt")
    old = f"{g.nx}x{g.ny}x{g.nz}/{g.n_views}x{g.nv}x{g.nu} 1 1\n"
    open(cache, "w").write(old)
    for _ in range(2):  # the second reads what the first appended
        batch = kct.Batch([geometry(g)])
        batch.tune(cache=cache)
        batch.close()
        lines = _lines(cache)
        assert open(cache).read().startswith(old) and len(lines) == 2
        assert lines[1][0] != lines[0][0] and lines[1][1] in "1234" and lines[1][2] in "01"


def test_recorded_iteration_follows_the_tuned_forms(tmp_path):
    """Choices read between two solves that move instances to the other backprojection
    kernel, or into it and out of it again: the replayed graph has the kernels they need."""
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    descs = [_cube(48, 48, 48, 1.0, 9), _cube(64, 60, 70, 0.7, 11)]
    geoms = [geometry(g) for g in descs]
    bs = [torch.from_numpy(ki.random_projections(g, 3)).to(dev()).to(torch.float32) for g in descs]
    batch = kct.Batch(geoms)
    cache = str(tmp_path / "tune.txt")
    batch.tune(cache=cache)
    keys = [ln[0] for ln in _lines(cache)]
    assert len(keys) == 2
    first = None
    for shapes in ((0, 0), (1, 0), (1, 1), (0, 1), (0, 0)):
        path = str(tmp_path / "pinned{}{}.txt".format(*shapes))
        open(path, "w").write("".join(f"{k} 1 {v}\n" for k, v in zip(keys, shapes)))
        batch.tune(cache=path)
        xs, infos = batch.cgls(bs, 4)
        xs = [x.clone() for x in xs]
        es, infos_e = batch.cgls(bs, 4, graph=False)
        first = first or xs
        for x, e, f, i, ie in zip(xs, es, first, infos, infos_e):
            assert torch.equal(x, e) and i.nr2 == ie.nr2 and i.iterations == 4
            assert rel(to_np(x), to_np(f)) < 1e-5
    batch.close()
