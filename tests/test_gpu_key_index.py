"""The key word's index field: a key's place among its record's keys, stored
in the bits between tile id and mask, or looked up where it does not fit."""
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


@pytest.mark.parametrize("box", [0, 1, 2])
def test_index_bits(R, box):
    """One plane of 32 x 32 tiles with records of 1 to 35 keys, alone (a wide
    index field) and beside 3,000 and 40,000 one-pixel planes that no Gaussian
    meets, which take all but 4 and all 16 of the field's bits: the same
    image, gradients and emission positions, bit for bit."""
    g = synth.make_gaussians(400, 41, (0, 0, 0.45), (1, 1, 0.55), (0.01, 0.3), aniso_max=4.0, opacity="random")
    base = synth.pack_planes([np.eye(3)], [(0.5, 0.5, 0.5)], [(1 / 200, 1 / 200)], [(200, 150)])
    dev = torch.device("cuda", 0)
    gd = R.to_device(g, dev)
    up = torch.from_numpy(np.random.default_rng(42).standard_normal(200 * 150).astype(np.float32)).to(dev)
    res = []
    for extra in (0, 3000, 40000):
        far = synth.pack_planes([np.eye(3)] * extra, [(0.5, 0.5, 1e3)] * extra, [(1.0, 1.0)] * extra,
                                [(1, 1)] * extra)
        pl = synth.Planes(*(np.concatenate([getattr(base, f), getattr(far, f)]) if extra else getattr(base, f)
                            for f in ("rot", "origin", "spacing", "wh")))
        plan = R.Plan(g.n, pl.wh, R.Params(tile_w=32, tile_h=32, box_mode=box), device=dev)
        pd = R.to_device(pl, dev)
        plan.fit(gd, pd)
        img = plan.render(gd, pd)
        grads = plan.backward(gd, pd, img, torch.cat([up, torch.zeros(extra, device=dev)]))
        key, eidx, rec, _ = plan.debug_keys()
        assert np.array_equal(np.sort(eidx), np.arange(key.size, dtype=np.uint32))
        per = np.bincount(rec)
        assert per.max() > 15 and plan.num_tiles == 35 + extra
        res.append((img[:200 * 150], grads, key, eidx, rec))
    for img, grads, key, eidx, rec in res[1:]:
        assert torch.equal(img, res[0][0])
        for a, b in zip(grads, res[0][1]):
            assert torch.equal(a, b)
        for a, b in zip((key, eidx, rec), res[0][2:]):
            assert np.array_equal(a, b)
