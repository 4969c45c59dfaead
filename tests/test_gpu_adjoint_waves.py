"""Adjoint accumulate with one wave per block (many tiles, few keys each) and
with four (the same scene with a larger key capacity): the sums of a key do not
depend on it, so the gradients are equal bit for bit; the loss is the float sum
of each tile's squared differences in another order."""
import numpy as np
import pytest

import oracle
from paper_2505_05643_amd import synth
from tests.parity import check_grads, oracle_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(8, 8), (16, 8), (8, 16), (16, 16), (32, 8), (32, 16), (16, 32), (32, 32)]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


def _run(R, g, pl, prm, cap, target):
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, prm, device=dev, key_capacity=cap)
    plan.fit(gd, pd)
    img = plan.render(gd, pd)
    loss = torch.zeros(1, device=dev)
    grads = plan.backward_mse(gd, pd, img, target, loss_buf=loss)
    return plan, img, grads, float(loss)


@pytest.mark.parametrize("tile", SHAPES)
@pytest.mark.parametrize("n", [40, 1500])
def test_waves_do_not_change_gradients(R, n, tile):
    """At least 1024 tiles: most empty (n = 40), or some tens of keys and, where
    the Gaussians crowd, more than one pass of a wave (n = 1500)."""
    g = synth.make_gaussians(n, 81, (0.3, 0.3, 0.3), (0.7, 0.7, 0.7), (0.01, 0.05), aniso_max=4.0, opacity="random")
    g.means[: n // 3] = 0.5 + 0.02 * (g.means[: n // 3] - 0.5)
    side = 33
    pl = synth.random_planes(2, 82, (8, 8), 1.0 / (side * max(tile)), 0.5, 0.5)
    pl.wh[:] = [[side * tile[0] - 3, side * tile[1] - 5]] * 2
    target = torch.from_numpy(np.random.default_rng(83).random(pl.npix).astype(np.float32)).cuda()
    prm = R.Params(tile_w=tile[0], tile_h=tile[1], box_mode=2)
    plan, img, one, la = _run(R, g, pl, prm, 0, target)
    px = tile[0] * tile[1]
    assert plan.num_tiles >= 1024
    assert (plan.key_capacity // plan.num_tiles) ** 2 * px < 3584 ** 2
    cap = plan.num_tiles * (int(3584 / px ** 0.5) + 2)
    plan4, img4, four, lb = _run(R, g, pl, prm, cap, target)
    assert torch.equal(img, img4)
    assert all(torch.equal(a, b) for a, b in zip(one, four))
    # a square passes at most 16 + 6 additions in its tile: 24 * 2^-24 each way
    assert abs(la - lb) <= 3e-6 * la


def test_one_wave_against_oracle(R):
    g = synth.make_gaussians(200, 84, (0.3, 0.3, 0.3), (0.7, 0.7, 0.7), (0.01, 0.05), aniso_max=4.0, opacity="random")
    pl = synth.random_planes(1, 85, (8, 8), 1 / 264, 0.5, 0.5)
    pl.wh[:] = [[264, 264]]
    prm = R.Params(tile_w=8, tile_h=8, box_mode=1)
    X = oracle.plane_points(pl)
    dimg = np.random.default_rng(86).standard_normal(pl.npix).astype(np.float32)
    _, _, k = oracle.ambiguity_points(g, X, oracle_params(prm))
    dimg[np.asarray(k).reshape(-1) > 0] = 0.0
    ref = oracle.grad_points(g, X, dimg.astype(np.float64), oracle_params(prm))
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, prm, device=dev)
    plan.fit(gd, pd)
    assert plan.num_tiles >= 1024
    img = plan.render(gd, pd)
    got = plan.backward(gd, pd, img, torch.from_numpy(dimg).to(dev))
    check_grads({k: t.cpu().numpy() for k, t in zip(("means", "lraw", "intensity", "opacity"), got)}, ref)
