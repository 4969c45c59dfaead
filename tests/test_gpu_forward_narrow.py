"""Forward on 8-wide tiles: a tile's records are evaluated four at a time, then
two, then one.  Every remainder, in the first round of a tile's records and in
a later one, against the oracle, with one and two waves per band."""
import numpy as np
import pytest

from paper_2505_05643_amd import synth
from tests.parity import check_image

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


@pytest.mark.parametrize("tile", [(8, 8), (8, 16)])
@pytest.mark.parametrize("split", [0, 1])
def test_remainders(R, tile, split):
    dev = torch.device("cuda", 0)
    for n in (1, 2, 3, 4, 5, 6, 7, 8, 63, 65, 66, 67, 131):
        # all over one tile and its neighbours
        g = synth.make_gaussians(n, 100 + n, (0.3, 0.3, 0.4), (0.7, 0.7, 0.6), (0.05, 0.2), opacity="random")
        pl = synth.random_planes(1, 101, (21, 19), 1 / 24, 0.5, 0.5)
        prm = R.Params(tile_w=tile[0], tile_h=tile[1], flags=R._lib.UG_FLAG_SPLIT_FORWARD if split else 0)
        gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
        plan = R.Plan(g.n, pl.wh, prm, device=dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        ranges = np.diff(plan.debug_keys()[3].astype(np.int64))
        assert ranges.max() > n // 2
        check_image(img.cpu().numpy(), g, pl, prm)
