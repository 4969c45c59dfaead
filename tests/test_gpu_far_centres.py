"""Records whose centre lies millions of pixels outside a plane that their
ellipse covers (a microscopic plane inside large Gaussians): no sub-block of
the plane may be left out, wherever the pixel distances stop being exact in
single precision (2^24)."""
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


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16), (32, 32)])
@pytest.mark.parametrize("spacing", [3e-8, 1e-8, 2e-9, 7e-10])
def test_microscopic_plane(R, tile, spacing):
    g = synth.make_gaussians(300, 91, (0, 0, 0), (1, 1, 1), (0.1, 0.4), opacity="random")
    pl = synth.random_planes(3, 92, (8, 8), spacing, 0.45, 0.55)
    pl.wh[:] = [[257, 21], [33, 65], [64, 40]]
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    for box in (0, 1, 2):
        prm = R.Params(tile_w=tile[0], tile_h=tile[1], box_mode=box)
        plan = R.Plan(g.n, pl.wh, prm, device=dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        assert plan.status() == 0
        recs = plan.debug_records()
        assert np.abs(recs["ub"]).max() > 2 ** 23 * (1e-8 / spacing)
        check_image(img.cpu().numpy(), g, pl, prm)
