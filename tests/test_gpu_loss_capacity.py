"""The loss of the fused mean-squared-error adjoint is the same bits whatever
key capacity the plan has (one or four waves per tile, one block per tile or
more)."""
import numpy as np
import pytest

from paper_2505_05643_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(8, 8), (16, 8), (8, 16), (16, 16), (32, 8), (32, 16), (16, 32), (32, 32)]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


@pytest.mark.parametrize("tile", SHAPES)
def test_loss_does_not_depend_on_the_capacity(R, tile):
    """More than 1024 tiles, ragged at the right and the bottom: few keys per
    tile (one wave), and room for 1,000 and 5,000 keys per tile."""
    g = synth.make_gaussians(400, 87, (0.3, 0.3, 0.3), (0.7, 0.7, 0.7), (0.01, 0.05), opacity="random")
    side = 33
    pl = synth.random_planes(2, 88, (8, 8), 1.0 / (side * max(tile)), 0.5, 0.5)
    pl.wh[:] = [[side * tile[0] - 3, side * tile[1] - 5]] * 2
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    rng = np.random.default_rng(89)
    losses = []
    for per_tile in (0, 1000, 5000):
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=tile[0], tile_h=tile[1], box_mode=2), device=dev)
        plan.fit(gd, pd)
        if per_tile:
            plan.reserve(plan.record_capacity, per_tile * plan.num_tiles)
        img = plan.render(gd, pd)
        if not losses:
            # targets that differ from the image in one tile only, so that the
            # other tiles' sums do not hide the rounding of that one
            W, H = int(pl.wh[0, 0]), int(pl.wh[0, 1])
            targets = []
            for tx, ty in rng.integers(0, side, size=(10, 2)):
                t = img.clone()
                view = t[:W * H].view(H, W)[ty * tile[1]:(ty + 1) * tile[1], tx * tile[0]:(tx + 1) * tile[0]]
                view += torch.from_numpy(rng.standard_normal(tuple(view.shape)).astype(np.float32)).to(dev)
                targets.append(t)
        out = []
        for t in targets:
            loss = torch.zeros(1, device=dev)
            plan.backward_mse(gd, pd, img, t, loss_buf=loss)
            out.append(float(loss))
        losses.append(out)
    exact = np.array([float(((img.double() - t.double()) ** 2).mean()) for t in targets])
    # the rounding of a difference counts twice, then at most 4 + 6 + 3
    # additions of one sign in float32 and the result's rounding
    assert np.all(np.abs(np.array(losses[0]) - exact) <= 16 * 2.0 ** -24 * exact)
    assert losses[1] == losses[0] and losses[2] == losses[0]
