"""Image-quality scores at the edges of the strips (64 input columns for 54
outputs) and row chunks: planes one pixel to either side of a strip, of a
chunk and of the window, alone (many chunks) and beside many others (one)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# both sides sum float64 moments of the same float32 pixels
TOL = 1e-9
WIDTHS = [1, 10, 11, 12, 63, 64, 65, 117, 118, 119, 173]
HEIGHTS = [1, 10, 11, 12, 13, 14, 15, 26, 27, 42, 43, 131]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


def _scores(R, wh, img, ref):
    dev = torch.device("cuda", 0)
    plan = R.Plan(1, wh, R.Params(), device=dev)
    s, m = plan.quality(torch.from_numpy(img).to(dev), torch.from_numpy(ref).to(dev))
    return s.cpu().numpy(), m.cpu().numpy()


def _check(R, wh, special=False):
    wh = np.asarray(wh, dtype=np.int32)
    rng = np.random.default_rng(61)
    npx = int(np.sum(wh[:, 0] * wh[:, 1]))
    img = rng.random(npx).astype(np.float32)
    ref = (img + 0.1 * rng.standard_normal(npx)).astype(np.float32)
    s, m = _scores(R, wh, img, ref)
    rs, rm = oracle.quality.quality(img, ref, wh, 1.0)
    assert np.array_equal(np.isnan(s), np.isnan(rs))
    ok = ~np.isnan(rs)
    assert np.all(np.abs(s[ok] - rs[ok]) <= TOL)
    np.testing.assert_allclose(m, rm, rtol=TOL, atol=0)


@pytest.mark.parametrize("w", WIDTHS)
def test_single_planes(R, w):
    for h in HEIGHTS:
        _check(R, [[w, h]])


def test_many_planes(R):
    _check(R, [[w, h] for w in WIDTHS for h in HEIGHTS] * 12)


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_pixel_stays_in_its_plane(R, value):
    """One such pixel: that plane's scores are NaN (the mean squared error of
    an infinity is infinite), the planes before and after keep theirs."""
    wh = np.array([[70, 40], [70, 40], [70, 40]], dtype=np.int32)
    rng = np.random.default_rng(62)
    img = rng.random(3 * 2800).astype(np.float32)
    ref = rng.random(3 * 2800).astype(np.float32)
    s0, m0 = _scores(R, wh, img, ref)
    img[2800 + 20 * 70 + 60] = value
    s, m = _scores(R, wh, img, ref)
    assert np.isnan(s[1]) and not np.isfinite(m[1])
    assert np.array_equal(s[[0, 2]], s0[[0, 2]]) and np.array_equal(m[[0, 2]], m0[[0, 2]])
