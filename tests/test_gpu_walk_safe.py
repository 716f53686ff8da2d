"""Cells through the walk tables' safe stretches (where a segment's own site is
taken without looking at the others) against the search over all sites."""
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


def _sites(layout, k, rng):
    if layout == "lattice":
        return scenes.make_sites("grid", 64)
    if layout == "twins":  # every site twice: exact ties, the lower index wins
        s = rng.uniform(-1.0, 1.0, ((k + 1) // 2, 3))
        return np.concatenate([s, s])[:k].astype(np.float32)
    if layout == "cluster":  # all within 2e-3: every site near everywhere
        return (0.2 + rng.uniform(-1e-3, 1e-3, (k, 3))).astype(np.float32)
    if layout == "line":
        return np.stack([np.linspace(-1.0, 1.0, k), 0.1 * np.ones(k), np.zeros(k)], 1).astype(np.float32)
    return rng.uniform(-1.0, 1.0, (k, 3)).astype(np.float32)


# 1, 2 and 4 lanes walk a ray from 2^19, 2^18 and no rays on
@pytest.mark.parametrize("layout,k,rays,n", [
    ("uniform", 17, 301, 193), ("uniform", 64, 5000, 64), ("uniform", 200, 700, 33),
    ("uniform", 40, 1 << 18, 4), ("uniform", 40, 1 << 19, 3), ("lattice", 64, 2000, 100),
    ("twins", 33, 900, 129), ("cluster", 30, 500, 64), ("line", 25, 500, 256)])
@pytest.mark.parametrize("near,far", [(0.0, 1.0), (2.0, 6.0)])
def test_safe_stretches_give_the_searched_cells(layout, k, rays, n, near, far):
    from paper_2011_12490_amd import derf
    rng = np.random.Generator(np.random.PCG64(rays + k))
    sites = _sites(layout, k, rng)
    k = len(sites)
    o = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    d = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    d[::7] *= 1e-4   # hardly moving: long stretches along a bisector
    d[1::7, 1:] = 0  # along an axis: in the lattice's bisector planes, along the line
    o[1::7, 1:] = 0.0
    d[5] = 0.0
    o[9], d[10], o[11, 0] = 1e30, 3e38, np.inf  # no nearest site in float32: the first
    o[12, 2] = np.nan
    r = derf.Renderer(sites, scenes.ARCH_TINY, scenes.make_weights(scenes.ARCH_TINY, k), "bf16")
    _, _, _, dbg = r.render(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), near, far, n,
                            seed=4, debug=True)
    torch.cuda.synchronize()
    t, cell = dbg["t"].cpu().numpy(), dbg["cell"].cpu().numpy()
    r.close()
    want = oracle.assign_depths(sites, o, d, t, nthreads=min(16, os.cpu_count() or 1))
    want = want[0] if isinstance(want, tuple) else want
    assert np.array_equal(cell, want)


@pytest.mark.parametrize("k,rays", [(17, 60), (40, 60), (23, 1 << 18), (23, 1 << 19)])
@pytest.mark.parametrize("layout", ["all_far", "some_far", "far_apart"])
def test_sites_beyond_float32_squares(layout, k, rays):
    """Sites whose squared distances overflow float32: with no finite distance
    the search takes the first site, and a ray's walk must not say otherwise."""
    from paper_2011_12490_amd import derf
    rng = np.random.Generator(np.random.PCG64(k + rays))
    sites = rng.uniform(-1.0, 1.0, (k, 3)).astype(np.float32)
    far = (np.sign(sites) * np.float32(2e19) + sites * np.float32(1e20)).astype(np.float32)
    if layout == "all_far":
        sites = far
    elif layout == "some_far":
        sites[::2] = far[::2]
    else:  # every distance is finite
        sites *= np.float32(1e18)
    o = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    d = rng.uniform(-1.0, 1.0, (rays, 3)).astype(np.float32)
    o[1] = np.float32(5e17)
    r = derf.Renderer(sites, scenes.ARCH_TINY, scenes.make_weights(scenes.ARCH_TINY, k), "bf16")
    dbg = r.render(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), 0.0, 1.0, 5, seed=4,
                   debug=True)[3]
    torch.cuda.synchronize()
    t, cell = dbg["t"].cpu().numpy(), dbg["cell"].cpu().numpy()
    r.close()
    want = oracle.assign_depths(sites, o, d, t, nthreads=min(16, os.cpu_count() or 1))
    want = want[0] if isinstance(want, tuple) else want
    assert np.array_equal(cell, want)
