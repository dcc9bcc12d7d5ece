"""The fixed-point form of the L1 scorer (GQE, LogicE), modelled in numpy on
the CPU: clamped query coordinates and what they were clamped by add up to the
distance; the largest sum does not wrap; and the error against 64 bits is below
that of the float sum where the table takes the form."""

import numpy as np
import pytest


def quantum_of(e, width):
    u_max = (2 ** 32 - 1) // width
    return np.nextafter(np.float32((float(e.max()) - float(e.min())) / u_max), np.float32(np.inf)), u_max


def words(x, lo, hi, q):
    c = np.clip(x, lo, hi)
    u = np.rint((c.astype(np.float64) - float(lo)) * (1.0 / float(q)))
    return u.astype(np.uint32), np.abs(x.astype(np.float64) - c.astype(np.float64)).sum(-1)


def takes_fixed(e, width):
    q, _ = quantum_of(e, width)
    mad = np.abs(e.astype(np.float64) - e.astype(np.float64).mean()).mean()
    return 0.41 * float(q) <= 0.25 * 0.25 * 2.0 ** -24 * width * mad


@pytest.mark.parametrize("width", [32, 100, 400, 513, 800, 8192])
def test_words_and_largest_sum(width):
    e = np.linspace(-3.0, 5.0, 1001).astype(np.float32)
    q, u_max = quantum_of(e, width)
    w, _ = words(e[:, None], e.min(), e.max(), q)
    assert w.min() == 0 and w.max() <= u_max
    assert u_max * width < 2 ** 32


@pytest.mark.parametrize("dist,width", [("uniform", 64), ("uniform", 400), ("normal", 400), ("uniform", 800)])
def test_error_below_the_float_sum(dist, width):
    g = np.random.default_rng(width)
    e = (g.uniform(-0.06, 0.06, (400, width)) if dist == "uniform" else g.normal(0, 0.02, (400, width))).astype(np.float32)
    qs = (e[:40] + g.uniform(-0.2, 0.2, (40, width))).astype(np.float32)
    assert takes_fixed(e, width)
    q, _ = quantum_of(e, width)
    we, _ = words(e, e.min(), e.max(), q)
    wq, ex = words(qs, e.min(), e.max(), q)
    ref = np.abs(qs[:, None].astype(np.float64) - e[None].astype(np.float64)).sum(-1)
    d = np.abs(wq[:, None].astype(np.int64) - we[None].astype(np.int64)).sum(-1)
    assert d.max() < 2 ** 32
    fixed = ex[:, None] + float(q) * d
    flt = np.zeros(ref.shape, np.float32)
    for k in range(width):
        flt += np.abs(qs[:, None, k] - e[None, :, k])
    err = lambda x: np.sqrt(np.mean((x - ref) ** 2))
    assert err(fixed) <= err(flt.astype(np.float64)), (err(fixed), err(flt))


def test_tables_that_keep_floats():
    g = np.random.default_rng(5)
    e = g.uniform(-0.5, 0.5, (300, 400)).astype(np.float32)
    assert takes_fixed(e, 400)
    e[0, 0] = 4000.0                                 # a range stretched by one value
    assert not takes_fixed(e, 400)
