"""Runs of records (the stretches of a record block that one wave builds): a
key's partial derivatives are placed by its run's offset.  Record counts at the
edges of waves, of blocks and of blocks of several rounds, on launches with and
without staged planes: the gradients of the launch are those of its planes
taken a few at a time."""
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


def _check(R, n, p, group, sigma):
    """Every Gaussian meets every plane: n p records."""
    g = synth.make_gaussians(n, 111, (0.1, 0.1, 0.499), (0.9, 0.9, 0.501), sigma, opacity="random")
    pl = synth.random_planes(p, 112, (24, 20), 1 / 20, 0.5, 0.5)
    pl.rot[:] = np.eye(3, dtype=np.float32).reshape(9)
    pl.origin[:] = np.stack([np.full(p, 0.5), np.full(p, 0.5), np.linspace(0.4995, 0.5005, p)], 1)
    dev = torch.device("cuda", 0)
    gd = R.to_device(g, dev)
    up = torch.from_numpy(np.random.default_rng(113).standard_normal((p, 480)).astype(np.float32)).to(dev)

    def grads(idx):
        sub = pl.subset(idx)
        pd = R.to_device(sub, dev)
        plan = R.Plan(n, sub.wh, R.Params(tile_w=8, tile_h=8, box_mode=1), device=dev)
        n_rec, _ = plan.fit(gd, pd)
        img = plan.render(gd, pd)
        return n_rec, plan.backward(gd, pd, img, up[idx].reshape(-1).contiguous())

    n_rec, whole = grads(np.arange(p))
    assert n_rec == n * p
    parts = None
    for a in range(0, p, group):
        _, x = grads(np.arange(a, min(a + group, p)))
        parts = [t.double() for t in x] if parts is None else [s + t.double() for s, t in zip(parts, x)]
    for a, b in zip(whole, parts):
        # float32 sums of p terms in another order
        assert float((a.double() - b).abs().max()) <= 2e-5 * float(b.abs().max())


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300])
def test_staged_planes(R, n):
    _check(R, n, 5, 2, (0.02, 0.1))


@pytest.mark.parametrize("n", [1, 7, 33])
def test_more_than_256_planes(R, n):
    _check(R, n, 300, 60, (0.02, 0.1))


@pytest.mark.parametrize("n,p", [(9000, 80), (9000, 140), (12000, 100)])
def test_blocks_of_several_rounds(R, n, p):
    """Two, three and three rounds of 256 records per block."""
    _check(R, n, p, 25, (0.003, 0.006))
