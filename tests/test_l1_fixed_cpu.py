"""The fixed-point form of the L1 scorer (GQE, LogicE): which tables take it
(the library's own rule, called on the host), and the arithmetic modelled in
numpy: clamped query coordinates and what they were clamped by add up to the
distance, the largest sum does not wrap, and the scores' error against 64 bits
beside that of the float form."""

import ctypes

import numpy as np
import pytest

from paper_2503_02172_amd import kgq


class L1Fixed(ctypes.Structure):
    _fields_ = [("on", ctypes.c_bool), ("lo", ctypes.c_float), ("hi", ctypes.c_float), ("quantum", ctypes.c_float)]


def choose(e, width, gamma, scale=1.0):
    """kgq::choose_l1_fixed(lo, hi, sum, width, gamma, scale)."""
    f = kgq.lib()._ZN3kgq15choose_l1_fixedEdddidd
    f.restype = L1Fixed
    f.argtypes = [ctypes.c_double] * 3 + [ctypes.c_int] + [ctypes.c_double] * 2
    return f(float(e.min()), float(e.max()), float(e.astype(np.float64).sum()), width, gamma, scale)


def words(x, f):
    c = np.clip(x, np.float32(f.lo), np.float32(f.hi))
    u = np.rint((c.astype(np.float64) - f.lo) * (1.0 / f.quantum)).astype(np.int64)
    return u, np.abs(x.astype(np.float64) - c.astype(np.float64)).sum(-1)


@pytest.mark.parametrize("width", [4, 32, 100, 400, 513, 800, 8192])
def test_words_and_largest_sum(width):
    e = np.linspace(-3.0, 5.0, 1001).astype(np.float32)
    f = choose(e, width, 1e6)
    assert f.on and f.lo == -3.0 and f.hi == 5.0
    u, ex = words(e[:, None], f)
    assert u.min() == 0 and u.max() * width < 2 ** 32 and not ex.any()


def scores(q, e, f, width, gamma, scale):
    """Scores of rows q against the same rows of e: fixed, float, 64 bits."""
    (uq, ex), (ue, _) = words(q, f), words(e, f)
    d = np.abs(uq - ue).sum(-1)
    assert d.max() < 2 ** 32
    fixed = ((gamma - scale * ex) - scale * float(f.quantum) * d.astype(np.float32).astype(np.float64)).astype(np.float32)
    acc = np.zeros(len(q), np.float32)
    for k in range(width):
        acc += np.abs(q[:, k] - e[:, k])
    flt = (gamma - scale * acc.astype(np.float64)).astype(np.float32)
    return fixed, flt, gamma - scale * np.abs(q.astype(np.float64) - e.astype(np.float64)).sum(-1)


def table(kind, width, gamma, g):
    """(entities, the usual spread of a coordinate)."""
    s = gamma / width
    if kind == "uniform":
        return g.uniform(-s, s, (500, width)), s
    if kind == "normal":
        return g.normal(0, s / 5, (500, width)), s / 5
    if kind == "bounds":
        return g.uniform(0, 1, (500, width)), 1.0
    if kind == "columns":                          # every column about its own centre
        return g.uniform(-1, 1, (1, width)) + 1e-3 * g.uniform(-1, 1, (500, width)), 1e-3
    if kind == "clusters":                         # tight groups of entities, far apart
        return g.uniform(-1, 1, (5, 1, width)).repeat(100, 1).reshape(500, width) + 1e-4 * g.uniform(-1, 1, (500, width)), 1e-4
    e = g.uniform(-s, s, (500, width))             # "outlier": a range stretched by one value
    e[3, 1] = 40.0
    return e, s


@pytest.mark.parametrize("kind,width,gamma,on", [
    ("uniform", 32, 12.0, True), ("uniform", 100, 24.0, True), ("uniform", 400, 24.0, True), ("uniform", 400, 1.0, True),
    ("uniform", 800, 24.0, False), ("normal", 400, 24.0, True), ("bounds", 800, 1.0, True), ("bounds", 800, 0.01, False),
    ("columns", 400, 24.0, False), ("columns", 400, 0.01, False), ("clusters", 64, 1.0, False), ("clusters", 400, 12.0, False),
    ("outlier", 400, 24.0, False), ("uniform", 400, 0.0, False)])
def test_rule_and_error_near_and_far(kind, width, gamma, on):
    """Tables take the form only where, however near the query is to the
    entity, the score's error stays within 4% of the float form's (3% from the
    rule, and the draw); over usual distances it is below that."""
    g = np.random.default_rng(width)
    scale = 1.0 / width if kind == "bounds" else 1.0
    e, spread = table(kind, width, gamma or 24.0, g)
    e = e.astype(np.float32)
    f = choose(e, width, gamma, scale)
    assert f.on == on
    if not on:
        return
    for near in (1.0, 1e-1, 1e-2, 1e-3, 1e-4, 1e-5):
        q = (e.repeat(8, 0) + near * spread * g.uniform(-1, 1, (4000, width))).astype(np.float32)
        fixed, flt, ref = scores(q, e.repeat(8, 0), f, width, gamma, scale)
        rms = lambda x: np.sqrt(np.mean((x.astype(np.float64) - ref) ** 2))
        assert rms(fixed) <= (1.0 if near == 1.0 else 1.04) * rms(flt), (near, rms(fixed), rms(flt))


def test_the_form_loses_near_entities_where_the_rule_refuses_it():
    """What the rule keeps out: a column-centred table at small gamma, in words
    of its range, is far coarser than its float sums."""
    g = np.random.default_rng(9)
    e, spread = table("columns", 400, 0.01, g)
    e = e.astype(np.float32)
    f = choose(e, 400, 1e6)
    assert f.on
    q = (e.repeat(8, 0) + 0.1 * spread * g.uniform(-1, 1, (4000, 400))).astype(np.float32)
    fixed, flt, ref = scores(q, e.repeat(8, 0), f, 400, 0.01, 1.0)
    assert np.sqrt(np.mean((fixed - ref) ** 2)) > 20 * np.sqrt(np.mean((flt - ref) ** 2))


def test_tables_that_keep_floats():
    e = np.full((300, 400), 0.25, np.float32)
    assert not choose(e, 400, 24.0).on                # one value: no range
    e[0, 0] = np.nan
    assert not choose(e, 400, 24.0).on
    e[0, 0] = np.inf
    assert not choose(e, 400, 24.0).on
