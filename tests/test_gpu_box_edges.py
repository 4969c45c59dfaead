"""Box support: the Eq. 13 box is decided in correctly rounded float64, so a
pixel centre exactly on its edge is inside and one an ulp beyond is not, also
where 1 / L lies so close to the middle of two doubles that a reciprocal that
is merely good to an ulp falls on the wrong side."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2505_05643_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BETA, CHI2 = np.float32(1e-4), np.float32(7.815)


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_05643_amd import raster
    return raster


def _hard(count):
    """Raw factor entries l whose 1 / (l^2 + beta) is nearest to a midpoint of
    two doubles, of three million seeded ones (boxes of about 1000 pixels)."""
    l = np.random.default_rng(17).uniform(0.048, 0.058, 3_000_000).astype(np.float32)
    L = l.astype(np.float64) ** 2 + np.float64(BETA)
    inv = 1.0 / L
    ulp = np.spacing(inv)
    off = np.abs(np.abs((np.longdouble(1) / L.astype(np.longdouble) - inv) / ulp) - 0.5)
    cand = np.argsort(off)[:4000]

    def distance(i):
        return abs(abs((1 / Fraction(float(L[i])) - Fraction(float(inv[i]))) / Fraction(float(ulp[i]))) - Fraction(1, 2))

    return l[sorted(cand, key=distance)[:count]]


def test_edges_on_hard_reciprocals(R):
    ls = np.unique(_hard(96))
    L = ls.astype(np.float64) ** 2 + np.float64(BETA)
    inv = 1.0 / L
    half = np.sqrt(np.float64(CHI2) * (inv * inv))
    n = ls.size
    wh, origin, means, own = [], [], [], []
    for i in range(n):
        W = int(round(2 * half[i])) + 1
        cu = 0.5 * W - 0.5
        for centre in (half[i], np.nextafter(half[i], np.inf)):
            m1 = centre - cu  # a multiple of half's ulp below a pixel: exact
            hi = np.float32(m1)
            lo = np.float32(hi.astype(np.float64) - m1)
            assert np.float64(hi) - np.float64(lo) == m1 and m1 + cu == centre
            means.append([hi, 0.0, 0.0])
            origin.append([lo, 0.0, 0.0])
            wh.append([W, 1])
            own.append(i)
    p = len(wh)
    pl = synth.Planes(np.tile(np.eye(3, dtype=np.float32).reshape(1, 9), (p, 1)),
                      np.asarray(origin, np.float32), np.ones((p, 2), np.float32), np.asarray(wh, np.int32))
    lraw = np.zeros((p, 6), np.float32)
    lraw[:, 0] = lraw[:, 3] = lraw[:, 5] = ls[own]
    g = synth.Gaussians(np.asarray(means, np.float32), lraw, np.full(p, 0.5, np.float32), np.ones(p, np.float32))
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    flags = R._lib.UG_FLAG_SCATTER | R._lib.UG_FLAG_BOX_SUPPORT
    plan = R.Plan(g.n, pl.wh, R.Params(flags=flags), device=dev)
    plan.fit(gd, pd)
    plan.render(gd, pd)
    recs = plan.debug_records()
    mine = recs[recs["gaussian"] == recs["plane"]]
    assert np.array_equal(mine["plane"], np.arange(p))
    first = mine["tx0"].reshape(n, 2)
    print("first pixel on the edge", np.bincount(first[:, 0], minlength=2), "beyond", np.bincount(first[:, 1], minlength=2))
    assert np.all(first[:, 0] == 0) and np.all(first[:, 1] == 1)
