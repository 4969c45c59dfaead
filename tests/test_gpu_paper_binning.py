"""PAPER boxes binned by rows: keys only for the tiles of the Eq. 13 box that
the ellipse reaches, while the counts and the capacity stay the box's."""
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


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 32), (16, 32)])
def test_paper_keys_are_the_reached_tiles(R, tile):
    """Needles and blobs on planes with cut tiles: the image and the gradients
    equal those of the tight binnings bit for bit, the emitted keys are a part
    of the box's tiles, measure and status count the whole box, and a capacity
    below that count is still an overflow."""
    tw, th = tile
    g = synth.make_gaussians(700, 31, (0, 0, 0), (1, 1, 1), (0.005, 0.03), aniso_max=30.0, opacity="random")
    pl = synth.random_planes(4, 32, (8, 8), 1 / 64, 0.3, 0.7)
    pl.wh[:] = [[77, 61], [64, 64], [9, 70], [1, 1]]
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    up = torch.from_numpy(np.random.default_rng(33).standard_normal(pl.npix).astype(np.float32)).to(dev)
    res = {}
    for bm in (0, 1, 2):
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=tw, tile_h=th, box_mode=bm), device=dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        res[bm] = (img, plan.backward(gd, pd, img, up), plan)
    for bm in (1, 2):
        assert torch.equal(res[0][0], res[bm][0])
        for a, b in zip(res[0][1], res[bm][1]):
            assert torch.equal(a, b)
    plan = res[0][2]
    recs = plan.debug_records()
    area = (recs["tx1"].astype(np.int64) - recs["tx0"] + 1) * (recs["ty1"].astype(np.int64) - recs["ty0"] + 1)
    box = int(np.maximum(area, 0).sum())
    emitted = plan.debug_keys()[0].size
    n_rec, n_key = plan.measure(gd, pd)
    assert n_key == box
    plan.render(gd, pd)
    assert plan.status(counts=True)[2] == box
    assert 0 < emitted <= box and (tile == (32, 32) or emitted < box)
    small = R.Plan(g.n, pl.wh, R.Params(tile_w=tw, tile_h=th), n_rec, box - 1, device=dev)
    img = small.render(gd, pd, torch.empty(pl.npix, device=dev), check_status=False)
    assert small.status() == R._lib.UG_ERR_CAPACITY and float(img.abs().max()) == 0.0
    print(tile, "box tiles", box, "emitted", emitted)
