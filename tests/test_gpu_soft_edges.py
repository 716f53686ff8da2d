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
                                     (33, 20), (63, 40), (64, 70), (65, 33), (130, 65)])
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
