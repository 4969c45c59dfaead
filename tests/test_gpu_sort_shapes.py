"""Sort of the keys by tile: small and large inputs (by key capacity), one pass
and two, at the tile counts where the digit widths change.  Every form gives
the stable order, so the sorted keys, the tile ranges and the image are equal
bit for bit, and equal to numpy's."""
import numpy as np
import pytest

from paper_2505_05643_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WIDE, SMALL = 512 * 1024, 1024 * 1024
# either side of the two lines by capacity, and 2048 blocks
CAPACITIES = [0, WIDE, WIDE + 1, SMALL, SMALL + 1, 2048 * 2048]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


@pytest.mark.parametrize("tiles", [(1, 1), (16, 16), (257, 1), (32, 32), (25, 41), (32, 64), (2049, 1), (64, 64), (241, 17), (257, 256)])
@pytest.mark.parametrize("n", [1, 300, 9000])
def test_sorted_keys(R, tiles, n):
    w, h = tiles[0] * 8, tiles[1] * 8
    g = synth.make_gaussians(n, 71, (0, 0, 0.45), (1, 1, 0.55), (0.01, 0.03), opacity="random")
    pl = synth.random_planes(1, 72, (8, 8), 1 / 64, 0.5, 0.5)
    pl.wh[:] = [[w, h]]
    pl.rot[:] = np.eye(3, dtype=np.float32).reshape(pl.rot[:].shape)
    pl.spacing[:] = 1.0 / max(w, h)
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    first = None
    for cap in CAPACITIES:
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=8, tile_h=8, box_mode=2), device=dev, key_capacity=cap)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        key, eidx, rec, ranges = plan.debug_keys()
        T = plan.num_tiles
        bits = max(1, int(np.ceil(np.log2(T))))
        tile = (key & ((1 << bits) - 1)).astype(np.int64)
        k = len(tile)
        assert k > 0 or n == 1
        assert np.array_equal(ranges, np.searchsorted(tile, np.arange(T + 1)))
        order = np.lexsort((eidx, tile))
        assert np.array_equal(order, np.arange(k)) and len(np.unique(eidx)) == k
        if first is None:
            first = (img, key, eidx, rec)
            continue
        assert torch.equal(first[0], img)
        assert np.array_equal(first[1], key) and np.array_equal(first[2], eidx) and np.array_equal(first[3], rec)
