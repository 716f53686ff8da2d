"""The precision of the float32 heads on the fp16 matrix units: their arithmetic
on the CPU (split_form.py) beside a float32 chain's, and the kernel's outputs
sample by sample against the float64 oracle."""
import os

import numpy as np
import pytest

import oracle
import split_form
from paper_2011_12490_amd import scenes

ARCHS = {"4x64": scenes.ARCH_TINY, "6x64": scenes.ARCH_SMALL, "8x128": scenes.ARCH_128}
# Largest error against float64 that float32 heads may show, per sample: rms of
# the densities over their own rms, rms of the colours (in [0, 1]).  Twice what
# the fp32 matrix units show on these heads and rays (5.6e-7 and 1.05e-7, 8x128
# at 40 units, most of it the encoding's angles).
SIGMA_RMS, RGB_RMS = 1.2e-6, 2.1e-7


def _weights(arch, kind, q, seed):
    """Glorot-uniform weights; bias: in every layer but the last a unit that the
    next layer does not read has a bias of 2^q; silent: one unit of every layer
    is 0 for every sample, and what reads it has weights 2^q times the others'."""
    w = scenes.make_weights(arch, 1, seed, 1.0)[0]
    v = scenes.weight_views(arch, w)
    if kind == "bias":
        for l in range(arch.depth - 1):
            v["hidden%d" % l][1][5] = 2.0 ** q
            c0 = arch.pos_dim if l + 1 == arch.skip_layer else 0
            v["hidden%d" % (l + 1)][0][:, c0 + 5] = 0.0
    if kind == "silent":
        for l in range(arch.depth):
            v["hidden%d" % l][0][3], v["hidden%d" % l][1][3] = 0.0, -1.0
            reads = ["hidden%d" % (l + 1)]
            if l + 1 == arch.depth:
                reads = ["sigma", "rgb_hidden" if arch.rgb_hidden else "rgb_out"]
            for t in reads:
                v[t][0][:, (arch.pos_dim if l + 1 == arch.skip_layer else 0) + 3] *= 2.0 ** q
    return w


CASES = [("plain", 0, 0.4), ("plain", 0, 40.0), ("bias", 4, 0.4), ("bias", 8, 0.4),
         ("silent", 8, 0.4), ("silent", 12, 0.4), ("silent", 16, 0.4), ("silent", 20, 0.4)]


def _rms(x, axis=None):
    return np.sqrt((np.asarray(x, np.float64) ** 2).mean(axis))


@pytest.mark.parametrize("arch", ARCHS)
@pytest.mark.parametrize("kind,q,scale", CASES)
def test_split_rounds_no_more_than_float32(arch, kind, q, scale):
    """The split form's outputs are no further from float64 than a float32
    chain's, for weights that fit it; without the low halves of the weights, or
    of the layers' entries, they miss the bars above."""
    a = ARCHS[arch]
    w = _weights(a, kind, q, 3)
    if not split_form.Scaled(a, w).fits:
        assert kind == "silent" and q > 8
        return
    rng = np.random.Generator(np.random.PCG64(5))
    x = rng.uniform(-scale, scale, (160, 3)).astype(np.float32)
    d = rng.normal(size=(160, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    ref = split_form.chain(a, w, x, d, np.float64)
    size = _rms(ref, 0)
    f32 = _rms(split_form.chain(a, w, x, d, np.float32) - ref, 0) / size
    got = _rms(split_form.split(a, w, x, d) - ref, 0) / size
    assert (got <= 1.1 * f32).all(), (got, f32)
    for lost in ({"low": False}, {"entries_low": False}):
        low = split_form.split(a, w, x, d, **lost) - ref
        assert _rms(low[:, 0]) > 4 * SIGMA_RMS * size[0]


@pytest.mark.gpu
@pytest.mark.parametrize("arch", ARCHS)
@pytest.mark.parametrize("kind,q,scale", CASES)
def test_float32_samples(arch, kind, q, scale):
    """Every sample's density and colour against the oracle at the bars above."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_12490_amd import derf
    a, heads, n = ARCHS[arch], 2, 64
    w = np.stack([_weights(a, kind, q, 30 + k) for k in range(heads)])
    sites = scenes.make_sites("uniform", heads)
    rng = np.random.Generator(np.random.PCG64(3))
    o = rng.uniform(-scale, scale, (64, 3)).astype(np.float32)
    d = rng.uniform(-0.5, 0.5, (64, 3)).astype(np.float32)
    ref = oracle.render(sites, a, w, o, d, 0.0, 1.0, n, 0, seed=6, per_sample=True,
                        nthreads=min(16, os.cpu_count() or 1))
    r = derf.Renderer(sites, a, w, "fp32")
    dbg = r.render(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), 0.0, 1.0, n, seed=6,
                   debug=True)[3]
    torch.cuda.synchronize()
    r.close()
    sigma = _rms(dbg["sigma"].cpu().numpy() - ref.sigma) / _rms(ref.sigma)
    rgb = _rms(dbg["rgb"].cpu().numpy() - ref.srgb)
    print("%s %s %d x%g: sigma %.2e rgb %.2e" % (arch, kind, q, scale, sigma, rgb))
    assert sigma <= SIGMA_RMS and rgb <= RGB_RMS
