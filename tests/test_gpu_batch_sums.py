"""A batched solve returns the separate solve's scalars to the bit, the residual norm
NR2 of the backprojection's partial sums among them, whatever the number of wavefronts
a brick's view subsets are dealt to, and in the workgroup bricks."""
import pytest

import kct_inputs as ki
from tests.gpu_util import dev, geometry, say, torch_mod
from tests.plan_util import BWD_BRICKS, BWD_DEEP, plan_of
from tests.test_gpu_forms import FORMS, _cube

pytestmark = pytest.mark.gpu

GEOMETRIES = {
    "depth_4": [FORMS["4x16"], FORMS["4x16_rows_chunked"]],
    "depth_8": [FORMS["8x16"], FORMS["8x8"]],
    "depth_16": [FORMS["16x16"], FORMS["16x8"], _cube(49, 41, 65, 1.0, 40)],
    "depth_32": [FORMS["32x4"]],
    "few_views": [_cube(49, 41, 51, 1.7, 1), _cube(49, 41, 51, 1.2, 2), _cube(49, 41, 65, 1.0, 3), _cube(33, 29, 21, 3.0, 5),
                  _cube(125, 123, 121, 0.7, 2)],
    "bricks": [_cube(131, 129, 115, 1.25, 1), _cube(161, 159, 163, 1.25, 2)],
    "deep_bricks": [_cube(256, 256, 256, 0.7, 1)],
}


@pytest.mark.parametrize("depth", sorted(GEOMETRIES))
def test_batch_scalars_equal_separate_solves(depth):
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    descs = GEOMETRIES[depth]
    geoms = [geometry(g) for g in descs]
    bs = [torch.from_numpy(ki.random_projections(g, 7)).to(dev()).to(torch.float32) for g in descs]
    for g in descs:
        if "bricks" in depth:
            assert plan_of(g)["form"] == {"bricks": BWD_BRICKS, "deep_bricks": BWD_DEEP}[depth]
    batch = kct.Batch(geoms)
    for K in (1, 2, 5):
        xs, infos = batch.cgls(bs, K)
        for g, b, x, i in zip(geoms, bs, xs, infos):
            x1, i1 = kct.cgls(g, b, K)
            say(f"[batch sums] {depth} K {K} vol {g.vol_shape}: nr2 {i.nr2!r} {i1.nr2!r}")
            assert torch.equal(x, x1)
            assert (i.nr2, i.nb, i.nb0) == (i1.nr2, i1.nb, i1.nb0)
    batch.close()


def test_small_batch_does_not_wait_for_its_queues():
    """Two 24^3 instances, 12 views: an iteration takes 0.26 ms; a draw from each of eight
    empty queues by every workgroup that the device holds made it 0.84 (bound: half way)."""
    import time
    import paper_2110_13526_amd as kct
    torch = torch_mod()
    descs = [_cube(24, 24, 24, 1.0, 12), _cube(24, 24, 24, 1.0, 12)]
    geoms = [geometry(g) for g in descs]
    bs = [torch.from_numpy(ki.random_projections(g, 7)).to(dev()).to(torch.float32) for g in descs]
    batch = kct.Batch(geoms)
    batch.cgls(bs, 4)
    best = float("inf")
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        batch.cgls(bs, 50)
        best = min(best, (time.perf_counter() - t) / 50)
    say(f"[batch sums] two 24^3 instances: {1e3 * best:.3f} ms per iteration")
    assert best < 0.55e-3
    batch.close()
