"""Sort of inputs whose blocks walk several rounds: the two round sizes, by keys
per block, with whole and part rounds."""
import numpy as np
import pytest

from paper_2505_05643_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


# mean keys per block of 2048 blocks on either side of 12288, and a second
# capacity that takes the other size for the same keys
@pytest.mark.parametrize("n,other", [(3400, 26_000_000), (8_200, 24_000_000)])
def test_several_rounds(R, n, other):
    g = synth.make_gaussians(n, 111, (0.1, 0.1, 0.48), (0.9, 0.9, 0.52), (0.03, 0.05), opacity="random")
    pl = synth.pack_planes([np.eye(3)], [(0.5, 0.5, 0.5)], [(1 / 2048, 1 / 2048)], [(2048, 2048)])
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    sides = set()
    first = None
    for cap in (0, other):
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=8, tile_h=8, box_mode=2), device=dev, key_capacity=cap)
        plan.fit(gd, pd)
        plan.render(gd, pd)
        assert plan.status() == 0
        key, eidx, rec, ranges = plan.debug_keys()
        sides.add(plan.key_capacity // 2048 >= 12288)
        tile = (key & 0xffff).astype(np.int64)
        assert plan.num_tiles == 1 << 16 and len(tile) > 2048 * 2048
        assert np.all(np.diff(tile << 32 | eidx.astype(np.int64)) > 0)
        assert np.array_equal(ranges, np.searchsorted(tile, np.arange(plan.num_tiles + 1)))
        by_emission = np.empty_like(rec)
        by_emission[eidx] = rec
        assert np.all(np.diff(by_emission.astype(np.int64)) >= 0)
        if first is None:
            first = (key, rec)
        else:
            assert np.array_equal(first[0], key) and np.array_equal(first[1], rec)
        del plan
    print("keys", len(first[0]), "sizes", sides)
    assert sides == {False, True}
