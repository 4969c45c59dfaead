"""The adjoint accumulate's per-pixel inputs and loss sums, formed per tile: cut
tiles, tiles without keys, and several blocks on one tile (only the first adds
to the loss)."""
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
@pytest.mark.parametrize("kind", ["none", "few", "many"])
def test_fused_mse_equals_separate(R, kind, tile):
    """Gradients bit for bit those of the separate loss gradient and adjoint;
    the loss within the rounding of a float sum over one tile: a pixel's square
    passes at most 4 + 6 + 3 additions and two roundings, 15 * 2^-24 < 1e-6."""
    if kind == "many":  # some thousand keys on each tile
        g = synth.make_gaussians(6000, 51, (0.3, 0.3, 0.3), (0.7, 0.7, 0.7), (0.2, 0.4), opacity="random")
    else:
        lo = 0.4 if kind == "few" else 40.0  # far from every plane: no record
        g = synth.make_gaussians(30, 52, (lo,) * 3, (lo + 0.2,) * 3, (0.01, 0.03), opacity="random")
    pl = synth.random_planes(4, 53, (8, 8), 1 / 48, 0.4, 0.6)
    pl.wh[:] = [[45, 37], [1, 50], [33, 9], [64, 64]]
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, R.Params(tile_w=tile[0], tile_h=tile[1], box_mode=2), device=dev)
    plan.fit(gd, pd)
    img = plan.render(gd, pd)
    target = torch.from_numpy(np.random.default_rng(54).random(pl.npix).astype(np.float32)).to(dev)
    _, d_image = R.mse_grad(img, target)
    want = plan.backward(gd, pd, img, d_image)
    loss = torch.zeros(1, device=dev)
    got = plan.backward_mse(gd, pd, img, target, loss_buf=loss)
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    exact = float(((img.double() - target.double()) ** 2).mean())
    assert abs(float(loss) - exact) <= 1e-6 * exact
