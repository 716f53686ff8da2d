"""The soft composite at the edges of its forms: heads around a wave, around the
staged table's limit and around a batch of loads; samples around a chunk."""
import os

import numpy as np
import pytest

import oracle
from paper_2011_12490_amd import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


@pytest.mark.parametrize("contrib", [True, False])
@pytest.mark.parametrize("heads,n", [(1, 1), (2, 64), (7, 65), (8, 63), (9, 128), (16, 129),
                                     (33, 20), (57, 21), (58, 22), (59, 64), (62, 30),
                                     (63, 40), (64, 70), (65, 33), (130, 65)])
def test_soft_heads_and_samples(heads, n, contrib):
    """Against the oracle at the float32 bar of 1e-4; heads 1, 4, 7, .. empty."""
    from paper_2011_12490_amd import derf
    arch, rays = scenes.ARCH_TINY, 9
    rng = np.random.Generator(np.random.PCG64(heads * 1000 + n))
    sites = rng.uniform(-1.0, 1.0, (heads, 3)).astype(np.float32)
    w = scenes.make_weights(arch, heads, sigma_bias=2.0)
    o = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    d = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    empty = np.arange(heads) % 3 == 1
    ref = oracle.render(sites, arch, w, o, d, 0.0, 1.0, n, 0, seed=3, mode="soft", beta=12.0,
                        contrib=True, empty=empty, nthreads=min(16, os.cpu_count() or 1))
    r = derf.Renderer(sites, arch, w, "fp32")
    r.set_empty_heads(list(empty))
    got = r.render_soft(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), 0.0, 1.0, n, 12.0,
                        seed=3, contrib=contrib)
    torch.cuda.synchronize()
    r.close()
    want = (ref.rgb, ref.depth, ref.opacity, ref.contrib)
    assert len(got) == (4 if contrib else 3)
    for x, y in zip(got, want):
        assert np.abs(x.cpu().numpy() - y).max() <= 1e-4


@pytest.mark.parametrize("heads", [3, 64, 65])
def test_soft_ignores_its_neighbours(heads):
    """Rays of NaN, infinite and huge origins leave the other rays' outputs
    bitwise as they are without them, and are not numbers themselves where a
    sample has no finite distance to any site."""
    from paper_2011_12490_amd import derf
    rng = np.random.Generator(np.random.PCG64(heads))
    sites = rng.uniform(-1.0, 1.0, (heads, 3)).astype(np.float32)
    r = derf.Renderer(sites, scenes.ARCH_TINY, scenes.make_weights(scenes.ARCH_TINY, heads, sigma_bias=2.0),
                      "bf16")
    o = rng.uniform(-1.0, 1.0, (40, 3)).astype(np.float32)
    d = rng.uniform(-1.0, 1.0, (40, 3)).astype(np.float32)
    bad = o.copy()
    bad[3], bad[11, 1], bad[12], bad[25] = np.nan, np.inf, 1e30, -3e38
    a, b = ([x.cpu().numpy() for x in r.render_soft(
        torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), 0.0, 1.0, 70, 12.0, seed=2,
        contrib=True)] for x in (o, bad))
    r.close()
    odd = [3, 11, 12, 25]
    keep = [i for i in range(40) if i not in odd]
    for x, y in zip(a, b):
        assert np.array_equal(x[keep], y[keep]) and np.isfinite(x).all()
        assert np.isnan(y[odd]).all()
