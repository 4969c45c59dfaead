"""Emission and record adjoint at the edges of their launch-size rules: a plan
fitted to its scene takes the forms for few records, the same scene with a
larger record capacity the ones for many, and both add and write in the same
order, so keys, image and gradients are equal bit for bit."""
import numpy as np
import pytest

from paper_2505_05643_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# record capacities around the rules' lines (128 and 512 record blocks of 256)
CAPACITIES = [32_768, 32_769, 131_072, 131_073, 1_200_000]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


@pytest.mark.parametrize("box_mode", [0, 1, 2])
@pytest.mark.parametrize("n,sigma,wh", [
    (1, (0.2, 0.3), [[64, 64]]),                       # one record
    (13, (0.5, 0.9), [[150, 90], [70, 120], [8, 8]]),  # few records of several hundred keys each
    (700, (0.02, 0.05), [[77, 61], [64, 64], [9, 70]]),
    (4000, (0.003, 0.006), [[64, 64]] * 6),            # about one key per record, whole and part waves
])
def test_capacity_does_not_change_results(R, n, sigma, wh, box_mode):
    g = synth.make_gaussians(n, 41, (0.4, 0.4, 0.4), (0.6, 0.6, 0.6), sigma, aniso_max=4.0, opacity="random")
    pl = synth.random_planes(len(wh), 42, (8, 8), 1 / 64, 0.45, 0.55)
    pl.wh[:] = wh
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    up = torch.from_numpy(np.random.default_rng(43).standard_normal(pl.npix).astype(np.float32)).to(dev)
    prm = R.Params(tile_w=8, tile_h=8, box_mode=box_mode)
    first = None
    for cap in [0] + CAPACITIES:
        plan = R.Plan(g.n, pl.wh, prm, device=dev, record_capacity=cap)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        grads = plan.backward(gd, pd, img, up)
        keys = plan.debug_keys()
        assert plan.status() == 0 and len(keys[0]) > 0
        if first is None:
            first = (img, grads, keys)
            continue
        assert torch.equal(first[0], img)
        assert all(torch.equal(a, b) for a, b in zip(first[1], grads))
        assert all(np.array_equal(np.asarray(a), np.asarray(b)) for a, b in zip(first[2], keys))
