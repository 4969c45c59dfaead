"""Adjoint accumulate at the edges of its work split: tiles with no key, a few
and many (several passes of a block, several blocks per tile), keys that reach
every column strip of a tile (more items than a wave's slots), thin ellipses
crossing many tiles, planes whose last tiles are cut, and no cut-off."""
import math

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


def _scene(kind):
    """(Gaussians, planes): ``few`` leaves most tiles empty, ``wide`` covers
    every pixel of the planes with every Gaussian, ``thin`` has needles."""
    if kind == "few":
        g = synth.make_gaussians(60, 11, (0, 0, 0), (1, 1, 1), (0.01, 0.03), opacity="random")
    elif kind == "wide":
        g = synth.make_gaussians(900, 12, (0.3, 0.3, 0.3), (0.7, 0.7, 0.7), (0.4, 0.9), opacity="random")
    else:
        g = synth.make_gaussians(500, 13, (0.2, 0.2, 0.2), (0.8, 0.8, 0.8), (0.004, 0.02), aniso_max=40.0,
                                 opacity="random")
    pl = synth.random_planes(3, 14, (8, 8), 1 / 48, 0.4, 0.6)
    pl.wh[:] = [[45, 37], [1, 50], [33, 9]]
    return g, pl


@pytest.mark.parametrize("kind,chi2", [("few", 7.815), ("wide", 7.815), ("thin", 7.815), ("thin", math.inf)])
def test_adjoint_tile_shapes(R, kind, chi2):
    """Every tile shape against the oracle's analytic gradient.  Pixels with a
    pair on the cut-off within rounding get no upstream gradient (which of the
    two they take is not defined); the tolerance is the parity tests'."""
    g, pl = _scene(kind)
    X = oracle.plane_points(pl)
    rng = np.random.default_rng(15)
    dimg = rng.standard_normal(pl.npix).astype(np.float32)
    prm = R.Params(chi2=chi2, box_mode=2)
    if math.isfinite(chi2):
        _, _, k = oracle.ambiguity_points(g, X, oracle_params(prm))
        dimg[np.asarray(k).reshape(-1) > 0] = 0.0
        assert np.count_nonzero(dimg) > 0.3 * dimg.size
    ref = oracle.grad_points(g, X, dimg.astype(np.float64), oracle_params(prm))
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    up = torch.from_numpy(dimg).to(dev)
    for tw, th in SHAPES:
        plan = R.Plan(g.n, pl.wh, R.Params(chi2=chi2, box_mode=2, tile_w=tw, tile_h=th), device=dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        first = plan.backward(gd, pd, img, up)
        again = plan.backward(gd, pd, img, up)
        for a, b in zip(first, again):
            assert torch.equal(a, b), "the adjoint is deterministic"
        out = {n: v.cpu().numpy().astype(np.float64) for n, v in zip(("means", "lraw", "intensity", "opacity"), first)}
        print(kind, chi2, (tw, th), "keys/tile", plan.status(counts=True)[2] / plan.num_tiles, check_grads(out, ref))


def test_adjoint_nan_upstream_stays_with_its_pixels(R):
    """A NaN in the upstream gradient reaches only the Gaussians whose support
    comes near that pixel: the rows an item is padded with are not read."""
    g = synth.make_gaussians(300, 21, (0, 0, 0.49), (1, 1, 0.51), (0.004, 0.02), opacity="random")
    pl = synth.pack_planes([np.eye(3)], [(0.5, 0.5, 0.5)], [(1 / 96, 1 / 96)], [(96, 96)])
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    for tw, th in ((16, 16), (32, 32)):
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=tw, tile_h=th), device=dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        up = torch.ones(pl.npix, device=dev)
        clean = plan.backward(gd, pd, img, up)
        at = int(img.argmax())  # a pixel some Gaussian covers
        up[at] = math.nan
        grads = plan.backward(gd, pd, img, up)
        bad = torch.isnan(grads.means).any(dim=1).cpu().numpy()
        near = np.hypot(g.means[:, 0] * 96 - (at % 96 + 0.5), g.means[:, 1] * 96 - (at // 96 + 0.5))
        assert bad.any() and np.all(near[bad] < 0.02 * 96 * math.sqrt(7.815) + 12)
        ok = torch.from_numpy(~bad).to(dev)
        for a, b in zip(clean, grads):
            assert torch.equal(a[ok], b[ok])
