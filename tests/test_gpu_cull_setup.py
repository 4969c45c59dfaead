"""Plane set-up inside the cull (few planes) and by its own kernel (65 planes
or more, or groups to search): the images agree bit for bit, and non-finite
inputs and overflows are reported either way, and only for that render."""
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


def _planes(p, extra=0):
    """p seeded planes and ``extra`` ones far from every Gaussian."""
    pl = synth.random_planes(p + extra, 91, (24, 17), 1 / 24, 0.3, 0.7)
    pl.origin[p:] += 1000.0
    return pl


@pytest.mark.parametrize("p", [1, 2, 7, 8, 9, 33, 64])
@pytest.mark.parametrize("n", [1, 63, 500, 40_000])
def test_setup_forms_agree(R, p, n):
    g = synth.make_gaussians(n, 92, (0, 0, 0), (1, 1, 1), (0.02, 0.06), opacity="random")
    dev = torch.device("cuda", 0)
    gd = R.to_device(g, dev)
    images = []
    for extra in (0, 65):
        pl = _planes(p, extra)
        pl.rot[:p], pl.origin[:p] = _planes(p).rot, _planes(p).origin
        pd = R.to_device(pl, dev)
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=8, tile_h=8), device=dev)
        plan.fit(gd, pd)
        images.append(plan.render(gd, pd)[: p * 24 * 17].clone())
        assert plan.status() == 0
    assert torch.equal(images[0], images[1])


@pytest.mark.parametrize("p", [1, 5, 64])
@pytest.mark.parametrize("n", [1, 700])
def test_bad_inputs_are_reported(R, p, n):
    g = synth.make_gaussians(n, 93, (0, 0, 0), (1, 1, 1), (0.2, 0.4), opacity="random")
    pl = _planes(p)
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, R.Params(tile_w=8, tile_h=8), device=dev)
    plan.fit(gd, pd)
    good = plan.render(gd, pd).clone()
    assert plan.status() == 0
    img = torch.empty_like(good)
    bad = R.GaussianTensors(*(t.clone() for t in gd))
    bad.means[n - 1, 1] = float("nan")
    plan.render(bad, pd, img, check_status=False)
    assert plan.status() == R._lib.UG_ERR_NONFINITE
    badp = R.PlaneTensors(*(t.clone() for t in pd))
    badp.origin.view(-1)[3 * (p - 1)] = float("inf")
    plan.render(gd, badp, img, check_status=False)
    assert plan.status() == R._lib.UG_ERR_NONFINITE
    recs = plan.status(counts=True)[1]
    plan.render(gd, pd, img, check_status=False)
    assert plan.status() == 0 and torch.equal(img, good)
    if n > 1:
        small = R.Plan(g.n, pl.wh, R.Params(tile_w=8, tile_h=8), device=dev, record_capacity=n // 2, key_capacity=64)
        small.render(gd, pd, img, check_status=False)
        assert small.status() == R._lib.UG_ERR_CAPACITY
        assert small.status(counts=True)[1] >= recs
