"""The packed 16-bit inverse YCoCg-R of the colour kernels, restated in numpy,
against the 32-bit definition (Sec. 4: t = Y - (Cg >> 1), G = Cg + t,
B = t - (Co >> 1), R = B + Co, each clamped to 0..255): every combination of the
16-bit edge values, each variable over its whole range at edge values of the
others, and random triples.
"""
import numpy as np


def sat(x):
    return np.clip(x, -32768, 32767)


def fits(x):
    assert x.min() >= -32768 and x.max() <= 32767
    return x


def packed(y, co, cg):
    h, k = cg >> 1, co >> 1
    g = sat(y + fits(cg - h))
    b = sat(y - fits(h + k))
    r = sat(y - fits(h - fits(co - k)))
    return [np.clip(c, 0, 255) for c in (r, g, b)]


def exact(y, co, cg):
    t = y - (cg >> 1)
    g = cg + t
    b = t - (co >> 1)
    return [np.clip(c, 0, 255) for c in (b + co, g, b)]


def check(y, co, cg):
    y, co, cg = (np.asarray(a, dtype=np.int64) for a in np.broadcast_arrays(y, co, cg))
    for p, e in zip(packed(y, co, cg), exact(y, co, cg)):
        assert np.array_equal(p, e)


def test_packed_colour_conversion_is_exact():
    edges = np.array([-32768, -32767, -16385, -16384, -16383, -257, -256, -255, -2, -1, 0, 1, 2, 127, 128, 254, 255, 256,
                      257, 511, 16383, 16384, 16385, 32766, 32767])
    full = np.arange(-32768, 32768)
    check(*np.meshgrid(edges, edges, edges))
    for a in edges:
        check(full[:, None], a, edges[None, :])
        check(a, full[:, None], edges[None, :])
        check(edges[None, :], a, full[:, None])
    r = np.random.default_rng(1)
    check(*r.integers(-32768, 32768, (3, 2_000_000)))
    check(*r.integers(-600, 900, (3, 2_000_000)))
