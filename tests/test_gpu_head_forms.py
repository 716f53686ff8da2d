"""Which form float32 heads take (derf_head_arithmetic), and the fp32 matrix
units' form through every render that can reach it: plain, hierarchical, soft,
culled in pieces, the stored encoding, and beside split heads."""
import os

import numpy as np
import pytest

import oracle
from paper_2011_12490_amd import scenes
from test_gpu_mlp_forms import _head, _rays

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ARCHS = {"4x64": scenes.ARCH_TINY, "6x64": scenes.ARCH_SMALL, "8x128": scenes.ARCH_128}
NTHREADS = min(16, os.cpu_count() or 1)
TOL = 1e-4  # the float32 bar


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    torch.cuda.set_device(0)


def _close(got, want):
    torch.cuda.synchronize()
    for x, y in zip(got, want):
        assert np.abs(x.cpu().numpy() - y).max() <= TOL


def _forms(derf, r, heads):
    return [derf.derf_head_arithmetic(r.handle, k) for k in range(heads)]


@pytest.mark.parametrize("arch", ARCHS)
@pytest.mark.parametrize("kind", ["plain", "small_units", "large_units", "dead", "tiny_row",
                                  "huge_bias"])
def test_form_of_the_heads(arch, kind):
    """One head decides for its architecture; bf16 heads have one form."""
    from paper_2011_12490_amd import derf
    a = ARCHS[arch]
    w = np.stack([_head(a, kind if k == 1 else "plain", 40 + k) for k in range(3)])
    sites = scenes.make_sites("uniform", 3)
    want = derf.DERF_ARITH_FP32 if kind in ("tiny_row", "huge_bias") else derf.DERF_ARITH_SPLIT
    r = derf.Renderer(sites, a, w, "fp32")
    assert _forms(derf, r, 3) == [want] * 3
    for k in (-1, 3):
        with pytest.raises(derf.DerfError) as e:
            derf.derf_head_arithmetic(r.handle, k)
        assert e.value.status == derf.DERF_ERR_INVALID_ARG
    r.close()
    r = derf.Renderer(sites, a, w, "bf16")
    assert _forms(derf, r, 3) == [derf.DERF_ARITH_BF16] * 3
    r.close()


@pytest.mark.parametrize("arch", ARCHS)
def test_every_render_on_the_fp32_units(arch):
    from paper_2011_12490_amd import derf
    a, heads, n, rays = ARCHS[arch], 5, 61, 45
    w = np.stack([_head(a, "tiny_row" if k == 2 else "plain", 60 + k) for k in range(heads)])
    sites = scenes.make_sites("uniform", heads)
    o, d = _rays(rays, seed=4)
    go, gd = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    r = derf.Renderer(sites, a, w, "fp32")
    assert _forms(derf, r, heads) == [derf.DERF_ARITH_FP32] * heads
    ref = oracle.render(sites, a, w, o, d, 0.0, 1.0, n, 0, seed=6, nthreads=NTHREADS)
    want = (ref.rgb, ref.depth, ref.opacity)
    plain = r.render(go, gd, 0.0, 1.0, n, seed=6)
    _close(plain, want)
    for levels, piece in ((3, 0), (6, 16), (3, 40)):  # (no ray gets near eps: nothing stops)
        *got, ev = r.render_culled(go, gd, 0.0, 1.0, n, 1e-9, levels, seed=6, piece=piece)
        _close(got, want)
        assert int(ev.min()) == n
    soft = oracle.render(sites, a, w, o, d, 0.0, 1.0, n, 0, seed=6, mode="soft", beta=9.0,
                         contrib=True, nthreads=NTHREADS)
    _close(r.render_soft(go, gd, 0.0, 1.0, n, 9.0, seed=6, contrib=True),
           (soft.rgb, soft.depth, soft.opacity, soft.contrib))
    # fine samples: at the depths that the library drew
    *got, dbg = r.render(go, gd, 0.0, 1.0, 20, 30, seed=6, debug=True)
    torch.cuda.synchronize()
    fine = oracle.render_depths(sites, a, w, o, d, 0.0, 1.0, dbg["t"].cpu().numpy(),
                                nthreads=NTHREADS)
    _close(got, (fine.rgb, fine.depth, fine.opacity))
    if a.skip_layer < 0:
        r.set_encoding(True)
        stored = r.render(go, gd, 0.0, 1.0, n, seed=6)
        torch.cuda.synchronize()
        for x, y in zip(plain, stored):
            assert torch.equal(x, y)
    r.close()


def test_one_architecture_of_a_mixed_renderer_on_the_fp32_units():
    from paper_2011_12490_amd import derf
    names = ["4x64", "6x64", "8x128", "6x64", "4x64", "8x128"]
    archs = [ARCHS[x] for x in names]
    w = [_head(a, "tiny_row" if k == 3 else "plain", 80 + k) for k, a in enumerate(archs)]
    sites = scenes.make_sites("uniform", len(archs))
    r = derf.Renderer(sites, archs, w, "fp32")
    assert _forms(derf, r, len(archs)) == [derf.DERF_ARITH_FP32 if x == "6x64" else
                                           derf.DERF_ARITH_SPLIT for x in names]
    o, d = _rays(70, seed=9)
    ref = oracle.render(sites, archs, w, o, d, 0.0, 1.0, 50, 0, seed=2, nthreads=NTHREADS)
    _close(r.render(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), 0.0, 1.0, 50, seed=2),
           (ref.rgb, ref.depth, ref.opacity))
    r.close()
