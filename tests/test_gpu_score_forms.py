"""The regrouped forms of the vector scorers where they could go wrong,
against the CPU oracle, at tolerances derived from the forms."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2503_02172_amd import synth
from tests.parity import check_scores, check_topk
from tests.test_split_f16_cpu import scale_of, split2

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
S = synth.STRUCTURE_ID


def _scores(w, model, structure, qb, k, center_reg=0.02, max_batch=None):
    import torch
    from paper_2503_02172_amd import kgq
    w.center_reg = center_reg
    with kgq.engine_for(w, max_batch=max_batch or qb.batch) as eng:
        out = eng.execute(S[structure], qb.anchors, qb.relations, k=k, scores=True)
        torch.cuda.synchronize()
        return {n: t.cpu().numpy() for n, t in out.items()}


@pytest.mark.parametrize("center_reg", [0.0, 0.02, 1.0])
@pytest.mark.parametrize("structure,B", [("1p", 37), ("2u", 5), ("1p", 1100)])
def test_gpu_cone_max_form(structure, B, center_reg):
    """ConE's one-term form of the weighted outside and inside distance at
    both ends of center_reg, in the small and the large row form, on cones of
    every aperture and axes up to +-pi (large output weights drive the
    projection's tanh to both ends, where cos(theta / 2) or cos(psi / 2)
    vanishes). Tolerance: per coordinate the distance is off by the angles'
    (a few ulp of pi: tanh, then half-angle sine and cosine) and products'
    rounding, at most 16 ulp of 1, then the sum's d ulp."""
    w = synth.make_tiny(O.CONE, n_ent=300, n_rel=7, dim=32, seed=61)
    w.params["proj.w3"] *= 12.0
    w.params["proj.b3"] *= 12.0
    d = w.dim
    w.params["entity.axis"][:4] = np.array([-np.pi, np.pi / 2, 0.0, -np.pi / 2], np.float32)[:, None]
    qb = synth.draw_queries(structure, B, 300, 7, seed=62)
    out = _scores(w, O.CONE, structure, qb, 5, center_reg)
    ref = O.Model(O.CONE, w.params, w.gamma, center_reg=center_reg).scores(S[structure], qb.anchors, qb.relations)
    mod = float(w.params["modulus"][0])
    # the projection's own float error moves its tanh inputs (12 times the
    # usual weights) by up to 12 * 4d ulp
    tol = 4 * EPS * abs(w.gamma) + mod * d * (16 + d + np.pi * 12 * 4 * d) * EPS
    assert np.abs(out["scores"] - ref).max() <= tol, (np.abs(out["scores"] - ref).max(), tol)


def _gqe(table, rel_scale, d, n_ent, seed):
    w = synth.make_tiny(O.GQE, n_ent=n_ent, n_rel=7, dim=d, seed=seed)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    if table == "normal":
        w.params["entity"] = rng.normal(0, 0.5, (n_ent, d)).astype(np.float32)
    elif table == "offset":
        w.params["entity"] += np.float32(100.0)
    elif table == "outlier":
        w.params["entity"][3, 1] = 4000.0
    elif table == "equal":
        w.params["entity"][:] = 0.25
    w.params["relation"] *= np.float32(rel_scale)
    return w


@pytest.mark.parametrize("table", ["uniform", "normal", "offset", "outlier", "equal"])
@pytest.mark.parametrize("d,B,rel_scale", [(32, 5, 1.0), (400, 9, 8.0), (100, 1100, 3.0), (8, 3, 1.0)])
def test_gpu_l1_fixed_and_float(table, d, B, rel_scale):
    """GQE's L1 scores on tables that take the fixed-point form (uniform,
    normal, shifted) and on those that keep floats (a far outlier, one value
    only), with query coordinates up to 24 times outside
    the table's range. Tolerance: every coordinate off by a quantum (range /
    2^23) and the state's two roundings, and the sum by width ulp."""
    n_ent = 300
    w = _gqe(table, rel_scale, d, n_ent, 71)
    qb = synth.draw_queries("3p", B, n_ent, 7, seed=72)
    out = _scores(w, O.GQE, "3p", qb, 5)
    ref = O.Model(O.GQE, w.params, w.gamma).scores(S["3p"], qb.anchors, qb.relations)
    e = w.params["entity"]
    rng = float(e.max() - e.min())
    dist = np.abs(w.gamma - ref)
    state = np.abs(e).max() + 3 * np.abs(w.params["relation"]).max()
    tol = d * (rng * 2.0 ** -23 + 4 * EPS * state) + (d + 4) * EPS * (dist + w.gamma)
    assert np.all(np.abs(out["scores"] - ref) <= tol), (np.abs(out["scores"] - ref) / tol).max()
    check_topk(out["idx"], out["score"], ref, 5, float((tol / np.maximum(np.abs(ref), w.gamma)).max()), w.gamma, table)


@pytest.mark.parametrize("n_ent,B", [(300, 40), (6000, 200), (3000, 1100)])
@pytest.mark.parametrize("kind,gamma", [("columns", 12.0), ("columns", 0.01), ("clusters", 0.5), ("uniform", 24.0)])
def test_gpu_l1_near_entities(kind, gamma, n_ent, B):
    """GQE's L1 scores where entities lie close together against the range of
    the whole table (columns of different centres, tight clusters), and on a
    table in fixed point: relations of zero, so a query is its anchor, exactly.
    Tolerance, root mean square over each query's nearest 30 entities: 1.1
    times what float32 sums and a float32 score leave, modelled in numpy."""
    d = 400
    g = np.random.Generator(np.random.PCG64(161))
    w = synth.make_tiny(O.GQE, n_ent=n_ent, n_rel=7, dim=d, seed=162, gamma=gamma)
    if kind == "columns":
        e = g.uniform(-1, 1, (1, d)) + 1e-3 * g.uniform(-1, 1, (n_ent, d))
    elif kind == "clusters":
        e = g.uniform(-1, 1, (n_ent // 50, 1, d)).repeat(50, 1).reshape(n_ent, d) + 1e-4 * g.uniform(-1, 1, (n_ent, d))
    else:
        e = g.uniform(-gamma / d, gamma / d, (n_ent, d))
    w.params["entity"] = e = e.astype(np.float32)
    w.params["relation"][:] = 0.0
    qb = synth.draw_queries("1p", B, n_ent, 7, seed=163)
    got = _scores(w, O.GQE, "1p", qb, 5)["scores"][:40]
    err, model = [], []
    for row, q in zip(got, e[qb.anchors[:40, 0]]):
        dist = np.abs(q.astype(np.float64) - e.astype(np.float64)).sum(1)
        at = np.argsort(dist)[:30]
        acc = np.zeros(30, np.float32)
        for k in range(d):
            acc += np.abs(q[k] - e[at, k])
        flt = (np.float64(w.gamma) - acc.astype(np.float64)).astype(np.float32)
        ref = w.gamma - dist[at]
        err.append(row[at] - ref)
        model.append(flt - ref)
    rms = lambda x: np.sqrt(np.mean(np.square(x)))
    assert rms(err) <= 1.1 * rms(model), (rms(err), rms(model))


@pytest.mark.parametrize("structure", ["2u", "pni", "1p"])
@pytest.mark.parametrize("B", [3, 700])
def test_gpu_l1_fixed_logice(structure, B):
    """LogicE's bounds in fixed point (width 2d = 128): union pairs, a
    negated answer path, single rows; split and unsplit scorers."""
    w = synth.make_tiny(O.LOGICE, n_ent=520, n_rel=7, dim=64, seed=81)
    qb = synth.draw_queries(structure, B, 520, 7, seed=82)
    out = _scores(w, O.LOGICE, structure, qb, 5)
    ref = O.Model(O.LOGICE, w.params, w.gamma).scores(S[structure], qb.anchors, qb.relations)
    # bounds in [0, 1]: a quantum of 2^-23, the states' own float error (three
    # dense layers of up to 4d terms, then a sigmoid), the mean's rounding
    tol = 2.0 ** -23 + 3 * 4 * 64 * EPS + 132 * EPS + 4 * EPS
    assert np.abs(out["scores"] - ref).max() <= tol, np.abs(out["scores"] - ref).max()


@pytest.mark.parametrize("bad", [np.inf, -np.inf])
def test_gpu_l1_infinite_query(bad):
    """A query state with an infinite coordinate is infinitely far from every
    entity in either form; other rows are untouched."""
    w = synth.make_tiny(O.GQE, n_ent=300, n_rel=7, dim=32, seed=91)
    w.params["relation"][2, 5] = bad
    qb = synth.draw_queries("1p", 8, 300, 7, seed=92)
    qb.relations[:, 0] = [0, 1, 2, 3, 4, 5, 6, 2]
    out = _scores(w, O.GQE, "1p", qb, 5)["scores"]
    assert np.all(np.isneginf(out[[2, 7]]))
    assert np.all(np.isfinite(np.delete(out, [2, 7], 0)))


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n_ent,B", [(6000, 200), (3000, 1100)])
def test_gpu_l1_not_finite_query_unsplit(n_ent, B, bad):
    """The same where the dimensions are not split (128 or more workgroups,
    small and large row form; d = 64 takes fixed point on this table): scores
    of -inf, ranked by index, or NaN; other rows are finite and untouched."""
    w = synth.make_tiny(O.GQE, n_ent=n_ent, n_rel=7, dim=64, seed=93)
    w.params["relation"][2, 5] = bad
    qb = synth.draw_queries("1p", B, n_ent, 7, seed=94)
    out = _scores(w, O.GQE, "1p", qb, 5)
    hit = qb.relations[:, 0] == 2
    assert hit.any()
    if np.isnan(bad):
        assert np.isnan(out["scores"][hit]).all()
    else:
        assert np.isneginf(out["scores"][hit]).all()
        assert np.array_equal(out["idx"][hit], np.tile(np.arange(5), (int(hit.sum()), 1)))
    assert np.isfinite(out["scores"][~hit]).all()


@pytest.mark.parametrize("model,name", [(O.GQE, "entity"), (O.Q2B, "entity"), (O.LOGICE, "entity.bounds")],
                         ids=["gqe", "q2b", "logice"])
@pytest.mark.parametrize("n_ent,d", [(70, 36), (257, 64), (64, 132)])
def test_gpu_point_table_layout_bf16(model, name, n_ent, d):
    """A bf16 entity table and its float32 values give the same scores (the
    re-layout's two input types, at ragged tiles of entities and coordinates)."""
    import torch
    from paper_2503_02172_amd import kgq
    w = synth.make_tiny(model, n_ent=n_ent, n_rel=7, dim=d, seed=95)
    bits = synth.bf16_rne(w.params[name])
    w.params[name] = synth.bf16_decode(bits)
    qb = synth.draw_queries("2i", 9, n_ent, 7, seed=96)
    outs = []
    for dtype in (kgq.F32, kgq.BF16):
        with kgq.Engine(model, n_ent, 7, d, w.gamma, 16, entity_dtype=dtype) as eng:
            for n, a in w.params.items():
                eng.load(n, bits if n == name and dtype == kgq.BF16 else a, dtype if n == name else kgq.F32)
            out = eng.execute(S["2i"], qb.anchors, qb.relations, k=5, scores=True)
            torch.cuda.synchronize()
            outs.append(out["scores"].cpu().numpy())
    assert np.array_equal(outs[0], outs[1])
    ref = O.Model(model, w.params, w.gamma).scores(S["2i"], qb.anchors, qb.relations)
    check_scores(outs[0], ref, w.rtol, w.gamma, name)


def _high_part(rows):
    """Rows with only the high f16 part of each value left."""
    s = np.array([scale_of(m) for m in np.abs(rows).max(1)])
    return np.stack([split2(r.astype(np.float32), q)[1] for r, q in zip(rows, s)]).astype(np.float64) * s[:, None]


def _uv(ab):
    """[U | V] of rows [a | b]."""
    from scipy.special import digamma
    a, b = np.split(ab, 2, 1)
    return np.concatenate([digamma(a + b) - digamma(a), digamma(a + b) - digamma(b)], 1)


@pytest.mark.parametrize("structure", ["1p", "2u", "pni"])
@pytest.mark.parametrize("n_ent,d,B,wide", [(300, 32, 5, False), (129, 36, 150, True), (1000, 52, 130, True),
                                           (64, 400, 33, True), (8200, 36, 260, False), (8200, 36, 530, False),
                                           (50100, 16, 3, False)])
def test_gpu_betae_split_scorer(structure, n_ent, d, B, wide):
    """BetaE's f16 matrix-core scorer at ragged entity and row tiles of all its
    forms, widths that end inside a 32-wide stage, and workgroups that take
    several tiles (of one stage each at d = 16); wide: entity parameters from
    1e-3 to 50 and query rows from 0.05 to 2^26 and 2^27, more than the 2^28
    that the form holds in full.

    The projections are the identity and every usual value a multiple of 2^-16,
    so the query rows are nearly the oracle's: large ones to 2^-23 for each of
    three layers, negated and averaged ones to three roundings. Tolerance: of
    the contraction C, whose terms are all positive, 2^-21 (the two operands'
    parts, and the dropped product) and 2^-24 for each stage's sum, and for the
    states' 10, the table's one and the scales' and sum's five; the states' part
    of C_q; what the form holds of a row's smallest values, 2^-50 of its largest;
    and the score's own rounding. A lost low part of either operand, planted
    here in the reference, is several times outside it."""
    import torch
    from paper_2503_02172_amd import kgq
    w = synth.make_tiny(O.BETAE, n_ent=n_ent, n_rel=7, dim=d, seed=101)
    rng = np.random.Generator(np.random.PCG64(102))
    p = w.params
    ab = p["entity.alpha_beta"]
    if wide:
        ab[:] = np.exp(rng.uniform(np.log(1e-3), np.log(50.0), ab.shape))
    ab[:] = np.maximum(np.round(ab * 2.0 ** 16), 1.0) * 2.0 ** -16
    rel = p["relation"]
    rel[:] = np.round(rel * 2.0 ** 16) * 2.0 ** -16
    if wide:
        spike = rng.random(rel.shape) < 0.02
        rel[spike] = np.round(rng.uniform(2.0 ** 21, 2.0 ** 22, spike.sum())) * 2.0 ** 4
        rel[rng.random(rel.shape) < 0.02] = -64.0          # to the regulariser's lower end
    for n in ("w1", "w2", "w3"):
        p["proj." + n][:] = np.eye(*p["proj." + n].shape)
    for n in ("b1", "b2"):
        p["proj." + n][:] = 0.0
    p["proj.b3"][:] = -1.0
    p["inter.w2"][:] = 0.0
    p["inter.b2"][:] = 0.0
    qb = synth.draw_queries(structure, B, n_ent, 7, seed=103)
    with kgq.engine_for(w, max_batch=B) as eng:
        eng.set_dense_path(kgq.DENSE_BF16X3)
        out = eng.execute(S[structure], qb.anchors, qb.relations, k=5, scores=True)
        torch.cuda.synchronize()
        got, idx, val = (out[n].cpu().numpy() for n in ("scores", "idx", "score"))
    m = O.Model(O.BETAE, p, w.gamma)
    ref = m.scores(S[structure], qb.anchors, qb.relations)
    uv = _uv(ab.astype(np.float64))
    terms = np.stack([m.query_states(S[structure], qa, qr) for qa, qr in zip(qb.anchors, qb.relations)])   # [B x terms x 2d]
    eps = (2.0 ** -21 + (-(-2 * d // 32) + 16) * EPS)
    tol = EPS * np.abs(ref)
    tol += np.max([eps * (t @ uv.T) + 10 * EPS * np.abs(t * _uv(t)).sum(1)[:, None] +
                   2.0 ** -50 * (t.max(1)[:, None] * uv.sum(1) + t.sum(1)[:, None] * uv.max(1))
                   for t in terms.transpose(1, 0, 2)], 0)
    assert np.all(np.abs(got - ref) <= tol), (np.abs(got - ref) / tol).max()
    check_topk(idx, val, got, 5, 0.0, w.gamma, structure)
    t, v = terms[:60, 0], uv[:500]
    c = t @ v.T
    for lost in (_high_part(t) @ v.T, t @ _high_part(v).T):
        assert (np.abs(lost - c) / (eps * c + EPS * np.abs(ref[:60, :500]))).max() > 4.0


@pytest.mark.parametrize("model", [O.BETAE, O.CONE, O.LOGICE], ids=["betae", "cone", "logice"])
@pytest.mark.parametrize("structure,d,B", [("2p", 32, 1), ("pni", 44, 16), ("2p", 36, 17), ("pni", 52, 32),
                                           ("pni", 36, 33), ("2p", 268, 32), ("2p", 52, 129), ("2p", 400, 512),
                                           ("2p", 400, 1990), ("2p", 128, 4100), ("2p", 128, 12289)])
def test_gpu_split_layers(model, structure, d, B):
    """Dense layers on rows in split form: every tile form (16 and 32 rows,
    one and two batches of K, the five tile shapes) at its edges, widths that
    end inside a 32-wide stage and outputs that end inside a tile. Every
    query's scores are as near to the oracle's as by layers on the FP32 matrix
    cores (1.5 times in the middle of the queries, 3 times at the worst, for the
    sums' other order); a lost low part of any layer's weights, planted here in
    the oracle, is not, by far."""
    w = synth.make_tiny(model, n_ent=70, n_rel=7, dim=d, seed=111)
    qb = synth.draw_queries(structure, B, 70, 7, seed=112)
    auto, fp32 = _auto_and_fp32(w, structure, qb)
    kw = {"center_reg": w.center_reg} if model == O.CONE else {}
    ref = O.Model(model, w.params, w.gamma, **kw).scores(S[structure], qb.anchors, qb.relations)
    check_scores(auto, ref, w.rtol, w.gamma, structure)
    per_query = lambda x, r: np.sqrt(np.mean(np.square(x - r), 1))
    err, base = per_query(auto, ref), per_query(fp32, ref)
    assert np.median(err) <= 1.5 * np.median(base) and err.max() <= 3.0 * base.max(), (np.median(err), np.median(base),
                                                                                       err.max(), base.max())
    few = slice(0, 64)
    layers = [n for n in w.params if n[-2] == "w" and (structure == "pni" or n.startswith("proj"))]
    for name in layers:
        lost = dict(w.params)
        lost[name] = _high_part(w.params[name]).astype(np.float32)
        seen = O.Model(model, lost, w.gamma, **kw).scores(S[structure], qb.anchors[few], qb.relations[few])
        assert np.median(per_query(seen, ref[few])) > 10.0 * np.median(base), name


def _auto_and_fp32(w, structure, qb, reverse=False):
    """Scores by the default paths and by the FP32 matrix cores; reverse: the
    parameters loaded last to first."""
    import torch
    from paper_2503_02172_amd import kgq
    outs = []
    if reverse:
        w.params = dict(reversed(w.params.items()))
    with kgq.engine_for(w, max_batch=qb.batch) as eng:
        for path in (kgq.DENSE_AUTO, kgq.DENSE_FP32):
            eng.set_dense_path(path)
            out = eng.execute(S[structure], qb.anchors, qb.relations, k=5, scores=True)
            torch.cuda.synchronize()
            outs.append(out["scores"].cpu().numpy())
    return outs


@pytest.mark.parametrize("model", [O.BETAE, O.CONE, O.LOGICE], ids=["betae", "cone", "logice"])
@pytest.mark.parametrize("layer,factor", [("proj.1", 2.0 ** 10), ("proj.1", 2.0 ** 28), ("proj.2", 2.0 ** 28)])
@pytest.mark.parametrize("B", [9, 200])
def test_gpu_split_layers_dominating_unit(model, layer, factor, B):
    """A hidden unit whose weights dwarf the others', switched off by its bias,
    leaves the scores' error against 64 bits where the FP32 matrix cores have
    it (half as much again for the sums' other order)."""
    w = synth.make_tiny(model, n_ent=70, n_rel=7, dim=64, seed=171)
    i = layer.rindex(".") + 1
    w.params[layer[:i] + "w" + layer[i:]][3] *= np.float32(factor)
    w.params[layer[:i] + "b" + layer[i:]].reshape(-1)[3] = -np.float32(factor) * 1000
    qb = synth.draw_queries("2p", B, 70, 7, seed=172)
    auto, fp32 = _auto_and_fp32(w, "2p", qb)
    kw = {"center_reg": w.center_reg} if model == O.CONE else {}
    ref = O.Model(model, w.params, w.gamma, **kw).scores(S["2p"], qb.anchors, qb.relations)
    rms = lambda x: np.sqrt(np.mean(np.square(x - ref)))
    assert rms(auto) <= 1.5 * rms(fp32), (rms(auto), rms(fp32))


@pytest.mark.parametrize("model", [O.BETAE, O.LOGICE], ids=["betae", "logice"])
@pytest.mark.parametrize("B,reverse", [(9, False), (200, True)])
@pytest.mark.parametrize("big", [2.0 ** 11, 2.0 ** 31])
def test_gpu_split_layers_wide_input_rows(model, B, reverse, big):
    """Layer inputs with one value far above the others (2^31: more than the
    2^28 that the form holds in full), and that value's weights as small: the
    scores' error against 64 bits stays where the FP32 matrix cores have it."""
    d = 64
    w = synth.make_tiny(model, n_ent=70, n_rel=7, dim=d, seed=181)
    col = 2 * d + 5 if model == O.LOGICE else 5
    w.params["relation"][:, 5] = np.linspace(0.5, 1.0, 7) * big
    w.params["proj.w1"][:, col] /= np.float32(big)
    qb = synth.draw_queries("2p", B, 70, 7, seed=182)
    auto, fp32 = _auto_and_fp32(w, "2p", qb, reverse)
    ref = O.Model(model, w.params, w.gamma).scores(S["2p"], qb.anchors, qb.relations)
    rms = lambda x: np.sqrt(np.mean(np.square(x - ref)))
    assert rms(auto) <= 1.5 * rms(fp32), (rms(auto), rms(fp32))


@pytest.mark.parametrize("d", [36, 64])
@pytest.mark.parametrize("name", ["inter.arg.w1", "inter.axis.w1", "inter.arg.b2"])
def test_gpu_cone_infinite_weight(name, d):
    """An infinite weight reaches what it feeds, as on the FP32 matrix cores:
    one of the aperture's does not touch the axis."""
    w = synth.make_tiny(O.CONE, n_ent=70, n_rel=7, dim=d, seed=173)
    w.params[name].reshape(-1)[5] = np.inf
    qb = synth.draw_queries("2i", 40, 70, 7, seed=174)
    auto, fp32 = _auto_and_fp32(w, "2i", qb)
    assert np.array_equal(auto, fp32, equal_nan=True)
    if name != "inter.axis.w1":
        assert np.isfinite(auto).all()


@pytest.mark.parametrize("n_ent,B,k", [(9001, 3, 1), (9001, 33, 70), (9001, 33, 71), (9001, 130, 64), (20011, 5, 156),
                                       (20011, 40, 157), (65600, 3, 256)])
@pytest.mark.parametrize("structure", ["1p", "2u"])
def test_gpu_topk_listed_small(structure, n_ent, B, k):
    """Top-k of small batches over a matrix with chunk keys, at both sides of
    two keys for each of the k and of the longest listed row (65,536), over
    entities in groups of eight equal ones (ties inside and across chunks):
    exactly the ranking of the returned scores, equal ones by index."""
    import torch
    from paper_2503_02172_amd import kgq
    w = synth.make_tiny(O.BETAE, n_ent=n_ent, n_rel=7, dim=16, seed=121)
    ab = w.params["entity.alpha_beta"]
    ab[:] = ab[(np.arange(n_ent) * 5 // 8) % n_ent]
    qb = synth.draw_queries(structure, B, n_ent, 7, seed=122)
    with kgq.engine_for(w, max_batch=B) as eng:
        eng.set_dense_path(kgq.DENSE_BF16X3)
        out = eng.execute(S[structure], qb.anchors, qb.relations, k=k, scores=True)
        torch.cuda.synchronize()
        got, idx, val = (out[n].cpu().numpy() for n in ("scores", "idx", "score"))
    want = np.argsort(-got, axis=1, kind="stable")[:, :k]
    assert np.array_equal(idx, want)
    assert np.array_equal(val, np.take_along_axis(got, want, 1))


@pytest.mark.parametrize("k", [1, 256, 257, 1024])
@pytest.mark.parametrize("n_ent,B", [(2049, 3), (4097, 64), (4096, 65), (8193, 5), (16384, 2), (16385, 33)])
def test_gpu_topk_few_rows(n_ent, B, k):
    """Register-resident top-k with 1,024 and with 256 threads a segment (at
    most 64 segments, and more) at the ends of its key counts, over few
    distinct scores: exactly the ranking of the returned scores."""
    import torch
    from paper_2503_02172_amd import kgq
    w = synth.make_tiny(O.GQE, n_ent=n_ent, n_rel=7, dim=8, seed=131)
    rng = np.random.Generator(np.random.PCG64(132))
    w.params["entity"][:] = rng.integers(0, 40, (n_ent, 8)).astype(np.float32) / 8
    qb = synth.draw_queries("1p", B, n_ent, 7, seed=133)
    out = _scores(w, O.GQE, "1p", qb, k)
    want = np.argsort(-out["scores"], axis=1, kind="stable")[:, :k]
    assert np.array_equal(out["idx"], want)
    assert np.array_equal(out["score"], np.take_along_axis(out["scores"], want, 1))


@pytest.mark.parametrize("every,sign", [(64, 1.0), (64, -1.0), (200, 1.0), (1, 1.0)])
@pytest.mark.parametrize("structure,B", [("1p", 3), ("2u", 130)])
def test_gpu_topk_listed_nan(structure, B, every, sign):
    """Top-k over a matrix with chunk keys in which whole entities score NaN:
    one in each chunk (more such chunks than k), one in about every third, and
    the first 300 entities. Exactly the ranking of the returned scores by their
    keys: NaNs by their bits, above +inf or below -inf, equal ones by index."""
    import torch
    from paper_2503_02172_amd import kgq
    n_ent, k = 9001, 64
    w = synth.make_tiny(O.BETAE, n_ent=n_ent, n_rel=7, dim=16, seed=141)
    bad = np.zeros(n_ent, bool)
    bad[: 300 if every == 1 else n_ent : every] = True
    w.params["entity.alpha_beta"][bad] = np.copysign(np.float32(np.nan), np.float32(sign))
    qb = synth.draw_queries(structure, B, n_ent, 7, seed=142)
    qb.anchors[:] = np.where(bad[qb.anchors], 8999, qb.anchors)
    with kgq.engine_for(w, max_batch=B) as eng:
        eng.set_dense_path(kgq.DENSE_BF16X3)
        out = eng.execute(S[structure], qb.anchors, qb.relations, k=k, scores=True)
        torch.cuda.synchronize()
        got, idx, val = (out[n].cpu().numpy() for n in ("scores", "idx", "score"))
    assert np.isnan(got[:, bad]).all() and np.isfinite(got[:, ~bad]).all()
    u = (got + np.float32(0.0)).view(np.uint32)
    key = np.where(u >> 31 != 0, ~u, u | np.uint32(0x80000000)).astype(np.int64)
    want = np.argsort(-key, axis=1, kind="stable")[:, :k]
    assert np.array_equal(idx, want)
    assert np.array_equal(val.view(np.uint32), np.take_along_axis(got, want, 1).view(np.uint32))


@pytest.mark.parametrize("model", [O.GQE, O.LOGICE], ids=["gqe", "logice"])
@pytest.mark.parametrize("n_ent,B", [(300, 30), (300, 1100), (6000, 200), (3000, 1100)])
def test_gpu_l1_fixed_row_position(model, n_ent, B):
    """One query at every position of a batch scores the same, bit for bit, in
    fixed point (width 64 takes it on these tables): split dimensions, small
    and large row form."""
    w = synth.make_tiny(model, n_ent=n_ent, n_rel=7, dim=64 if model == O.GQE else 32, seed=151)
    qb = synth.draw_queries("2p", B, n_ent, 7, seed=152)
    qb.anchors[:], qb.relations[:] = qb.anchors[:1], qb.relations[:1]
    out = _scores(w, model, "2p", qb, 5)
    assert np.array_equal(out["scores"], np.broadcast_to(out["scores"][:1], (B, n_ent)))
    assert np.array_equal(out["idx"], np.broadcast_to(out["idx"][:1], (B, 5)))
