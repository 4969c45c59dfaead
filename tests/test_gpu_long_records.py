"""Record adjoint of small launches: 64 records whose keys are spread evenly
are read by their own lanes, others are staged together.  Every form adds a
record's keys in emission order, so the gradients equal, bit for bit, those of
a plan with record capacity beyond the small launches'."""
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


def _grads(R, g, pl, prm, records):
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, prm, device=dev)
    plan.fit(gd, pd)
    if records:
        plan.reserve(records, plan.key_capacity)
    img = plan.render(gd, pd)
    up = torch.from_numpy(np.random.default_rng(96).standard_normal(pl.npix).astype(np.float32)).to(dev)
    keys = np.bincount(plan.debug_keys()[2])
    return plan.backward(gd, pd, img, up), keys


@pytest.mark.parametrize("n,big,lo,hi", [(70, 70, 0.3, 0.5),     # every record over the whole plane: even
                                         (64, 64, 0.02, 0.05),   # some tens of keys, uneven lengths
                                         (300, 4, 0.01, 0.02),   # a few long records among short ones: staged
                                         (200, 70, 0.01, 0.02),  # near the line
                                         (65, 1, 0.004, 0.005)])
def test_forms_agree(R, n, big, lo, hi):
    g = synth.make_gaussians(n, 97, (0.2, 0.2, 0.2), (0.8, 0.8, 0.8), (lo, hi), opacity="random")
    rng = np.random.default_rng(98)
    which = rng.permutation(n)[:big]
    if big < n:
        g.lraw[which] = 0.0
        for k in (0, 3, 5):
            g.lraw[which, k] = np.sqrt(1 / rng.uniform(0.1, 0.4, big)).astype(np.float32)
    pl = synth.random_planes(3, 99, (117, 101), 1 / 117, 0.45, 0.55)
    prm = R.Params(tile_w=8, tile_h=8, box_mode=2)
    small, keys = _grads(R, g, pl, prm, 0)
    large, _ = _grads(R, g, pl, prm, 64 * 2048 + 1)
    assert keys.max() > (8 if big > 1 else 1)
    assert all(torch.equal(a, b) for a, b in zip(small, large))
