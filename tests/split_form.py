"""The arithmetic of the float32 heads, in numpy: the form on the fp16 matrix
units (split operands), a float32 chain (the fp32 units) and float64.

Used on the CPU to say how the split form's rounding compares with float32's,
for which weights, and what a lost low half would show.  It repeats the
arithmetic (scales, splits, the three products and their fp32 sums), not the
kernel's layout.
"""
import numpy as np

from paper_2011_12490_amd import scenes

F = np.float32


def _frexp(x):
    return np.frexp(x)[1]


def encode(p, levels):
    """gamma of float32 points, rounded to float32 once."""
    q = p.astype(np.float64)
    out = [q]
    for l in range(levels):
        out += [np.sin(q * (np.pi * 2.0 ** l)), np.cos(q * (np.pi * 2.0 ** l))]
    return np.concatenate(out, 1).astype(F)


def _split(a):
    """a (float32, below 2^16) as two fp16 values, held in float64."""
    hi = a.astype(np.float16)
    lo = (a - hi.astype(F)).astype(np.float16)
    return hi.astype(np.float64), lo.astype(np.float64)


class Scaled:
    """A head's weights as the split form scales them (rows brought to the size
    of their layer's median row, stored times 2^shift), per-layer bounds;
    low=False drops the weights' low halves."""

    def __init__(self, arch, w, low=True):
        self.arch = arch
        v = {t: (m.copy(), b.copy()) for t, (m, b) in scenes.weight_views(arch, w.astype(F)).items()}
        tags = ["hidden%d" % l for l in range(arch.depth)]
        tags += ["rgb_hidden"] if arch.rgb_hidden else []

        self.fits = True  # (the rows' part of the rule)

        def exps(m):  # a row's scale to [1, 2), as an exponent
            u = np.abs(m)
            top = u.max(1)
            small = (u > 0) & (u < top[:, None] * F(2.0 ** -12))
            if (4 * small.sum(1) > (u > 0).sum(1)).any() or (np.abs(1 - _frexp(top)) > 40)[top > 0].any():
                self.fits = False
            return 1 - _frexp(top), top > 0

        self.shift = {"sigma": 14, "rgb_out": 14}
        last = "rgb_hidden" if arch.rgb_hidden else "rgb_out"
        for l, t in enumerate(tags):
            m, b = v[t]
            x, some = exps(m)
            k = np.sort(x[some])[some.sum() // 2] if some.any() else 0
            self.shift[t] = 14 + k
            f = np.where(some, np.ldexp(F(1), x - k), F(1)).astype(F)
            m *= f[:, None]
            b *= f
            if t == "rgb_hidden":
                reads = [("rgb_out", 0)]
            elif l + 1 == arch.depth:
                reads = [("sigma", 0), (last, 0)]
            else:
                reads = [(tags[l + 1], arch.pos_dim if l + 1 == arch.skip_layer else 0)]
            for r, c0 in reads:
                v[r][0][:, c0:c0 + len(f)] /= f
        self.factor = {}
        for t in ("sigma", "rgb_out"):
            x, some = exps(v[t][0])
            f = np.where(some, np.ldexp(F(1), x), F(1)).astype(F)
            v[t][0][:] *= f[:, None]
            self.factor[t] = 1 / f
        self.v = v
        self.bound = {t: (F(1.001) * np.abs(v[t][0]).sum(1, dtype=F).max(),
                          F(1.001) * np.abs(v[t][1]).max()) for t in tags}
        self.halves = {}
        for t, (m, _) in v.items():
            hi, lo = _split(np.ldexp(m, self.shift[t]))
            self.halves[t] = (hi, lo if low else 0 * lo)


def _mfma(acc, a, b):
    """acc += b a^T in chunks of 16 columns, rounded to fp32 after each."""
    return (acc.astype(np.float64) + b @ a.T).astype(F)


def _split_layer(halves, xs, low):
    """The three products of one layer, over the entries' scaled float32 values
    (low=False: without the entries' low halves)."""
    hi, lo = halves
    acc = np.zeros((len(xs), len(hi)), F)
    xh, xl = _split(xs)
    xl = xl if low else 0 * xl
    for k in range(0, xs.shape[1], 16):
        s = slice(k, k + 16)
        for a, b in ((lo[:, s], xh[:, s]), (hi[:, s], xl[:, s]), (hi[:, s], xh[:, s])):
            acc = _mfma(acc, a, b)
    return acc


def split(arch, w, x, d, low=True, entries_low=True):
    """(density before its ReLU, colour logits) [m, 4] of the split form; without
    the low halves of the weights or of the layers' entries."""
    s = Scaled(arch, w, low)
    gx, gd = encode(x, arch.pos_freqs), encode(d, arch.dir_freqs)
    in_max = np.maximum(1, np.abs(x).max(1)).astype(F)
    e = _frexp(in_max)

    def times(v, p):
        return (v * np.exp2(p.astype(np.float64))[:, None]).astype(F)

    h, m = times(gx, 15 - e), in_max

    def layer(tag, xs, e, m, least):
        n1, b1 = s.bound[tag]
        bound = np.maximum((n1 * m + b1).astype(F), least)
        ne = np.maximum(_frexp(np.minimum(bound, F(2.0 ** 126))), -100)
        acc = _split_layer(s.halves[tag], xs, entries_low)
        out = (acc.astype(np.float64) * np.exp2((e - ne - s.shift[tag]).astype(np.float64))[:, None] +
               times(np.broadcast_to(s.v[tag][1], acc.shape), 15 - ne)).astype(F)
        out = np.maximum(out, 0)
        return out, ne, np.ldexp(out.max(1), ne - 15).astype(F)

    for l in range(arch.depth):
        if l and l == arch.skip_layer:
            h, m = np.concatenate([times(gx, 15 - e), h], 1), np.maximum(m, in_max)
        least = in_max if l + 1 == arch.skip_layer else F(1) if l + 1 == arch.depth else F(0)
        h, e, m = layer("hidden%d" % l, h, e, m, least)

    def rows(tag, xs, e):
        acc = _split_layer(s.halves[tag], xs, entries_low)
        true = times(acc, e - 29)
        return (true.astype(np.float64) * s.factor[tag] + s.v[tag][1]).astype(F)

    sigma = rows("sigma", h, e)
    z = np.concatenate([h, times(gd, 15 - e)], 1)
    if arch.rgb_hidden:
        z, e, _ = layer("rgb_hidden", z, e, np.maximum(m, 1).astype(F), F(0))
    return np.concatenate([sigma, rows("rgb_out", z, e)], 1)


def chain(arch, w, x, d, dtype):
    """The same, in float64, or in float32 with a sum rounded term by term
    (from the bias on, as the fp32 units take it)."""
    v = scenes.weight_views(arch, w.astype(F))
    gx, gd = encode(x, arch.pos_freqs).astype(dtype), encode(d, arch.dir_freqs).astype(dtype)

    def dense(tag, z):
        m, b = v[tag]
        if dtype is np.float64:
            return z @ m.T.astype(dtype) + b
        acc = np.broadcast_to(b, (len(z), len(b))).astype(F)
        for k in range(z.shape[1]):
            acc = (acc.astype(np.float64) + z[:, k:k + 1].astype(np.float64) * m[None, :, k]).astype(F)
        return acc

    h = gx
    for l in range(arch.depth):
        if l and l == arch.skip_layer:
            h = np.concatenate([gx, h], 1)
        h = np.maximum(dense("hidden%d" % l, h), 0)
    sigma = dense("sigma", h)
    z = np.concatenate([h, gd], 1)
    if arch.rgb_hidden:
        z = np.maximum(dense("rgb_hidden", z), 0)
    return np.concatenate([sigma, dense("rgb_out", z)], 1)
