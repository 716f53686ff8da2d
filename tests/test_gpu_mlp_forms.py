"""The grouped MLP's tile queues at the edges of their range."""
import numpy as np
import pytest

from paper_2011_12490_amd import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _rays(count, seed=3):
    rng = np.random.Generator(np.random.PCG64(seed))
    o = rng.uniform(-1.0, 1.0, (count, 3)).astype(np.float32)
    d = rng.uniform(-0.5, 0.5, (count, 3)).astype(np.float32)
    return o, d


# 4x64 bf16 tiles hold 256 samples and three workgroups share a compute unit
# (256 of them): one to a few tiles, one short of and one past a tile per
# workgroup, and several per workgroup, where stretches run out and are
# stolen from
@pytest.mark.parametrize("tiles", [1, 3, 9, 766, 767, 768, 769, 775, 1537, 3000])
@pytest.mark.parametrize("heads", [1, 5])
def test_every_tile_is_taken_once(tiles, heads):
    """A frame equals its quarters rendered one by one, bitwise (a tile taken
    twice writes the same values, so the outputs are poisoned first)."""
    from paper_2011_12490_amd import derf
    n, rays = 64, 4 * tiles
    sites = scenes.make_sites("uniform", heads)
    r = derf.Renderer(sites, scenes.ARCH_TINY, scenes.make_weights(scenes.ARCH_TINY, heads, sigma_bias=1.0),
                      "bf16")
    o, d = (torch.from_numpy(x).cuda() for x in _rays(rays))
    # a first render of other rays leaves its own outputs in the workspace
    r.render(o.flip(0).contiguous(), d, 0.0, 1.0, n, seed=9)
    whole = r.render(o, d, 0.0, 1.0, n, seed=5)
    for q in range(4):
        a, b = q * tiles, (q + 1) * tiles
        part = r.render(o[a:b].contiguous(), d[a:b].contiguous(), 0.0, 1.0, n, seed=5, ray_offset=a)
        torch.cuda.synchronize()
        for x, y in zip(whole, part):
            assert torch.equal(x[a:b], y)
    r.close()
