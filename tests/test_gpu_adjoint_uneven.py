"""Adjoint accumulate where some tiles have far more keys than the mean: their
keys behind the dealt ones are found by chunks of the sorted list.  A key's
sums do not depend on who takes it, so the gradients equal, bit for bit, those
of a plan with room enough that every tile's own blocks take all its keys."""
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


def _scene(counts, tile, side, others):
    """counts[i] small Gaussians inside tile 3 + i of row 5 (in pixel units),
    and some anywhere, on one plane of side x side tiles."""
    tw, th = tile
    g = synth.make_gaussians(sum(counts) + others, 93, (0, 0, -0.5), (side * tw, side * th, 0.5), (1.0, 3.0),
                             opacity="random")
    at = 0
    for i, n in enumerate(counts):
        s = slice(at, at + n)
        g.means[s, 0] = (3 + i) * tw + tw / 2 + 0.3 * np.sin(np.arange(n))
        g.means[s, 1] = 5 * th + th / 2 + 0.3 * np.cos(np.arange(n))
        g.means[s, 2] = 0.0
        g.lraw[s] = 0.0
        g.lraw[s, 0] = g.lraw[s, 3] = g.lraw[s, 5] = np.sqrt(1 / 0.6)  # 2.8 standard deviations: 1.7 pixels
        at += n
    pl = synth.pack_planes([np.eye(3)], [(side * tw / 2, side * th / 2, 0.0)], [(1.0, 1.0)], [(side * tw, side * th)])
    return g, pl


def _grads(R, g, pl, tile, per_tile):
    dev = torch.device("cuda", 0)
    gd, pd = R.to_device(g, dev), R.to_device(pl, dev)
    plan = R.Plan(g.n, pl.wh, R.Params(tile_w=tile[0], tile_h=tile[1], box_mode=2), device=dev)
    plan.fit(gd, pd)
    if per_tile:
        plan.reserve(plan.record_capacity, per_tile * plan.num_tiles)
    img = plan.render(gd, pd)
    up = torch.from_numpy(np.random.default_rng(94).standard_normal(pl.npix).astype(np.float32)).to(dev)
    target = torch.from_numpy(np.random.default_rng(95).random(pl.npix).astype(np.float32)).to(dev)
    loss = torch.zeros(1, device=dev)
    a = plan.backward(gd, pd, img, up)
    b = plan.backward_mse(gd, pd, img, target, loss_buf=loss)
    ranges = plan.debug_keys()[3].astype(np.int64)
    return plan, list(a) + list(b) + [loss], np.diff(ranges)


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16), (32, 32)])
@pytest.mark.parametrize("counts", [(1024,), (1025, 2047), (1280, 3000, 1), (255, 1537, 4097), (9001,)])
def test_four_waves(R, tile, counts):
    """Few tiles: a tile's blocks take 1024 keys, the chunks have 256."""
    g, pl = _scene(counts, tile, 8, 60)
    _, got, per = _grads(R, g, pl, tile, 0)
    assert per.max() >= max(counts)
    plan, ref, _ = _grads(R, g, pl, tile, (int(per.max()) // 1024 + 1) * 1024)
    assert plan.key_capacity // plan.num_tiles >= per.max()
    assert all(torch.equal(x, y) for x, y in zip(got, ref))


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 32)])
@pytest.mark.parametrize("counts", [(256,), (257, 511), (320, 700, 1), (4097,)])
def test_one_wave(R, tile, counts):
    """At least 1024 tiles with few keys on average: a tile's block takes 256
    keys."""
    g, pl = _scene(counts, tile, 33, 300)
    plan, got, per = _grads(R, g, pl, tile, 0)
    assert per.max() >= max(counts) and plan.num_tiles >= 1024
    assert (plan.key_capacity // plan.num_tiles) ** 2 * tile[0] * tile[1] < 3584 ** 2
    _, ref, _ = _grads(R, g, pl, tile, (int(per.max()) // 1024 + 1) * 1024)
    assert all(torch.equal(x, y) for x, y in zip(got, ref))


def test_long_chunks(R):
    """Room for 2M keys, nearly all in three tiles: chunks of 1024."""
    counts = (70_001, 33_000, 120_000)
    g, pl = _scene(counts, (16, 16), 8, 60)
    dev = torch.device("cuda", 0)
    _, got, per = _grads(R, g, pl, (16, 16), 2_000_000 // 64)
    assert per.max() >= max(counts)
    _, ref, _ = _grads(R, g, pl, (16, 16), (int(per.max()) // 1024 + 1) * 1024)
    assert all(torch.equal(x, y) for x, y in zip(got, ref))
