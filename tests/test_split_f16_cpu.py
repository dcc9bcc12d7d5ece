"""The two-part f16 split behind the f16 matrix-core form, checked in numpy on
the CPU (no GPU code is run here).

Claims checked, for rows of float32 values scaled by the power of two that
brings the largest into [2^14, 2^15): with h = f16(x) and l = f16((x - h)
2048), x - h is exact in float32 and x = h + l / 2048 to 2^-23 of x down to
2^-28 of the row's largest value, and to 2^-50 of the largest below; the
three kept part products miss a product by less than 2^-21 of it; and the
contraction of rows of positive values, summed in float32 over stages of 32,
is no further from 64 bits than the six-product bf16 form's; nor is a chain of
dense layers further than float32's, from the dimensions on where the layers
take the form."""

import ctypes

import numpy as np
import pytest

from paper_2503_02172_amd import kgq

from tests.test_split_bf16_cpu import split3


def scale_of(m):
    e = (np.float32(m).view(np.uint32) >> 23) & 255
    if e == 0:
        return np.float32(2.0 ** -100)
    if e == 255:
        return np.float32(1.0)
    return np.array([max(int(e) - 14, 1) << 23], np.uint32).view(np.float32)[0]


def split2(x, s):
    y = (x.astype(np.float32) * (np.float32(1.0) / s)).astype(np.float32)
    h = y.astype(np.float16)
    r = (y - h.astype(np.float32)).astype(np.float32)
    return y, h, r, (r * np.float32(2048.0)).astype(np.float16)


@pytest.mark.parametrize("span", [0, 10, 28, 60])
def test_split_error(span):
    g = np.random.default_rng(span)
    for m in (1.0, 3e4, 1e-20, 2e30):
        x = (g.uniform(1, 2, 20000) * np.exp2(-g.integers(0, span + 1, 20000)) * g.choice([-1.0, 1.0], 20000) * m).astype(np.float32)
        big = np.abs(x).max()
        s = scale_of(big)
        assert 2.0 ** 14 <= float(big) / float(s) < 2.0 ** 15
        y, h, r, l = split2(x, s)
        assert np.array_equal(r.astype(np.float64), y.astype(np.float64) - h.astype(np.float64)), "x - h"
        err = np.abs(h.astype(np.float64) + l.astype(np.float64) / 2048 - y.astype(np.float64)) * float(s)
        assert np.all(err <= np.maximum(np.abs(x.astype(np.float64)) * 2.0 ** -23, float(big) * 2.0 ** -50))


def test_scale_is_a_finite_power_of_two():
    for m in (0.0, 1e-45, 1.2e-38, 1e-30, 1.0, 3.4e38, np.inf, np.nan):
        s = scale_of(np.float32(m))
        assert np.frexp(s)[0] == 0.5 and np.isfinite(np.float32(1.0) / s)


def test_three_products_bound():
    g = np.random.default_rng(3)
    x, y = (g.uniform(1, 2, 50000).astype(np.float32) for _ in range(2))
    (_, h, _, l), (_, H, _, L) = split2(x, scale_of(x.max())), split2(y, scale_of(y.max()))
    h, l, H, L = (v.astype(np.float64) for v in (h, l, H, L))
    kept = (h * H + (h * L + l * H) / 2048) * float(scale_of(x.max())) * float(scale_of(y.max()))
    ref = x.astype(np.float64) * y.astype(np.float64)
    assert np.all(np.abs(kept - ref) <= 2.0 ** -21 * ref)


@pytest.mark.parametrize("K", [64, 800])
def test_positive_contraction_no_further_off_than_bf16x3(K):
    g = np.random.default_rng(K)
    a = np.maximum(1 + g.uniform(-1, 1, (60, K)), 0.05).astype(np.float32)
    a[30:] = (1.0 / a[30:]).astype(np.float32)                # negated rows: reciprocals
    u = (g.gamma(0.7, 1.5, (200, K)) + 0.01).astype(np.float32)
    ref = a.astype(np.float64) @ u.astype(np.float64).T

    def staged(parts):
        """Sum over stages of 32: each product's stage in 64 bits (the matrix
        core's own sum), rounded into a float32 accumulator."""
        accs = [np.zeros(ref.shape, np.float32) for _ in range(max(p[2] for p in parts) + 1)]
        for k in range(0, K, 32):
            for p, q, i in parts:
                accs[i] = (accs[i] + p[:, k:k + 32].astype(np.float64) @ q[:, k:k + 32].astype(np.float64).T).astype(np.float32)
        return accs

    sa = np.array([scale_of(r.max()) for r in a])[:, None]
    su = np.array([scale_of(r.max()) for r in u])[:, None]
    ah, al = (np.stack([split2(r, s[0])[i] for r, s in zip(a, sa)]) for i in (1, 3))
    uh, ul = (np.stack([split2(r, s[0])[i] for r, s in zip(u, su)]) for i in (1, 3))
    hi, lo = staged([(ah, uh, 0), (ah, ul, 1), (al, uh, 1)])
    new = (hi + lo * np.float32(1 / 2048)) * (sa * su.T)
    (xh, xm, xl, _, _), (yh, ym, yl, _, _) = split3(a), split3(u)
    old = staged([(xh, yh, 0), (xh, ym, 0), (xm, yh, 0), (xm, ym, 0), (xh, yl, 0), (xl, yh, 0)])[0]
    rms = lambda x: np.sqrt(np.mean(((x.astype(np.float64) - ref) / ref) ** 2))
    assert rms(new) <= rms(old), (rms(new), rms(old))


def split_rows(x):
    s = np.array([scale_of(r) for r in np.abs(x).max(1)])
    parts = [split2(r, q) for r, q in zip(x, s)]
    return np.stack([p[1] for p in parts]).astype(np.float64), np.stack([p[3] for p in parts]).astype(np.float64), s


def layer(x, w, b, bounded, relu):
    """One layer on split rows x = (h, l, scale) as the kernel does it, its
    output in float32, or split again under the scale of its bound."""
    (xh, xl, xs), (wh, wl, ws) = x, split_rows(w)
    hi = np.zeros((len(xh), len(w)), np.float32)
    lo = hi.copy()
    for k in range(0, xh.shape[1], 32):
        s = slice(k, k + 32)
        hi = (hi + xh[:, s] @ wh[:, s].T).astype(np.float32)
        lo = (lo + xh[:, s] @ wl[:, s].T).astype(np.float32)
        lo = (lo + xl[:, s] @ wh[:, s].T).astype(np.float32)
    y = ((hi + lo * np.float32(1 / 2048)) * (xs[:, None] * ws[None]) + b).astype(np.float32)
    y = np.maximum(y, 0) if relu else y
    if not bounded:
        return y
    bound = xs * np.float32(32768) * np.abs(w).sum(1).max() + np.float32(max(b.max(), 0))
    s = np.array([scale_of(v) for v in bound])
    parts = [split2(r, q) for r, q in zip(y, s)]
    return np.stack([p[1] for p in parts]).astype(np.float64), np.stack([p[3] for p in parts]).astype(np.float64), s


def layer32(x, w, b, relu):
    acc = np.zeros((len(x), len(w)), np.float32)
    for k in range(0, x.shape[1], 4):                # v_mfma_f32_16x16x4_f32
        acc = (acc + x[:, k:k + 4].astype(np.float64) @ w[:, k:k + 4].T.astype(np.float64)).astype(np.float32)
    y = (acc + b).astype(np.float32)
    return np.maximum(y, 0) if relu else y


def projection(g, d, factors=(1.0, 1.0), big=1.0):
    """Errors of BetaE's three projection layers, (split, float32), with one
    unit of each hidden layer scaled by a factor and switched off, and one input
    value `big` times the others and its weights as small."""
    def make(o, i):
        lim = np.sqrt(6.0 / (o + i))
        return g.uniform(-lim, lim, (o, i)).astype(np.float32), (g.uniform(-1, 1, o) / np.sqrt(i)).astype(np.float32)
    x = (np.maximum(g.uniform(0, 2, (48, 2 * d)), 0.05) + g.uniform(-0.5, 0.5, (48, 2 * d))).astype(np.float32)
    ws = [make(4 * d, 2 * d), make(4 * d, 4 * d), make(2 * d, 4 * d)]
    x[:, 5] *= np.float32(big)
    ws[0][0][:, 5] /= np.float32(big)
    for (w, b), f in zip(ws, factors):
        if f > 1:
            w[3] *= np.float32(f)
            b[3] = -np.float32(f) * 1000
    ref, y32, y = x.astype(np.float64), x, split_rows(x)
    for i, (w, b) in enumerate(ws):
        ref = ref @ w.T.astype(np.float64) + b
        ref = np.maximum(ref, 0) if i < 2 else ref
        y32 = layer32(y32, w, b, i < 2)
        y = layer(y, w, b, i < 2, i < 2)
    n = np.linalg.norm
    return n(y - ref) / n(ref), n(y32 - ref) / n(ref)


@pytest.mark.parametrize("d", [32, 64, 200])
def test_layers_no_further_off_than_float32(d):
    g = np.random.default_rng(d)
    split, flt = np.mean([projection(g, d) for _ in range(6)], 0)
    assert split <= flt, (split, flt)


LIMIT = 16384.0                                      # kSplitSpreadMax


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("factors,big", [((LIMIT, 1.0), 1.0), ((1.0, LIMIT), 1.0), ((128.0, 128.0), 1.0),
                                         ((1.0, 1.0), LIMIT), ((16.0, 16.0), 64.0)])
def test_layers_with_a_value_far_above_the_others(d, factors, big):
    """At the largest spread that the form takes, with the unit that makes it
    switched off or the input value's weights as small, the layers are no
    further off than float32 ones (10% for the draw); at 2^24 they would be."""
    g = np.random.default_rng(d)
    split, flt = np.mean([projection(g, d, factors, big) for _ in range(4)], 0)
    assert split <= 1.1 * flt, (split, flt)
    more = 2.0 ** 24 / LIMIT
    f = [v * more if v == max(*factors, big) else v for v in (*factors, big)]
    split, flt = projection(g, d, tuple(f[:2]), f[2])
    assert split > 5 * flt


class SplitBound(ctypes.Structure):
    _fields_ = [("norm", ctypes.c_float), ("bias", ctypes.c_float), ("spread", ctypes.c_float), ("fits", ctypes.c_bool)]


def bound(sums, bias):
    """kgq::split_bound(sums, bias, n)."""
    f = kgq.lib()._ZN3kgq11split_boundEPKfS1_l
    f.restype = SplitBound
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long]
    sums = np.asarray(sums, np.float32)
    bias = None if bias is None else np.asarray(bias, np.float32)
    return f(sums.ctypes.data, None if bias is None else bias.ctypes.data, sums.size)


def test_split_bound():
    b = bound([3.0, 5.0, 4.0], [0.5, -100.0, -1.0])
    assert (b.norm, b.bias, b.fits) == (5.0, 0.5, True) and b.spread == np.float32(5.0 / 4.0)
    assert bound([3.0, 5.0, 4.0], None).bias == 0.0
    assert bound([3.0, 4096.0 * 4, 4.0], None).spread == 4096.0
    assert bound([3.0, 4.0, 4.0], [0.0, 1e6, 0.0]).spread > 1e5          # a huge positive bias counts,
    assert bound([3.0, 4.0, 4.0], [0.0, -1e6, 0.0]).spread == 1.0        # a negative one switches the unit off
    assert bound([0.0, 0.0, 4.0], None).spread == np.inf
    assert bound([0.0, 0.0], None).spread == 1.0
    for bad in (np.nan, np.inf, 2.0 ** 21):
        assert not bound([3.0, bad, 4.0], None).fits
    for bad in (np.nan, np.inf, -np.inf, 2.0 ** 41):
        assert not bound([3.0, 4.0], [0.0, bad]).fits


def test_table_spread():
    f = kgq.lib()._ZN3kgq12table_spreadEPKd
    f.restype = ctypes.c_float
    f.argtypes = [ctypes.c_void_p]

    def spread(rows):
        """rows: (largest magnitude, sum of log2, count) of a few workgroups."""
        p = np.zeros((512, 3))
        p[:len(rows)] = np.reshape(rows, (-1, 3))
        return f(p.ctypes.data)
    assert spread([]) == 1.0                                             # all zeros
    assert spread([(2.0, 0.0, 4), (8.0, 4.0, 4)]) == np.float32(8.0 / 2.0 ** 0.5)
    for bad in (np.nan, np.inf, -np.inf):
        assert spread([(2.0, bad, 4)]) == np.inf
    assert spread([(np.inf, 3.0, 4)]) == np.inf
