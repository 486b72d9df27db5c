"""logsumexp over infinite values: a fold with +inf among its terms is +inf, one
of -inf alone is -inf, in every form of the fold (dense pulls from marks and
from a list, short and long in-edge lists, hash-table accumulators, sorted
groups) and where terms of one key meet in different passes."""
import numpy as np
import pytest

from helpers import LSE_TOL, engine_run
from oracle import evaluate
from paper_2609_27203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched_rounds", [0, 4])
@pytest.mark.parametrize("sources", [1, 40, 64, 130])
def test_one_infinite_term_in_a_pull(sources, batched_rounds):
    """A target's terms from up to 20 middle nodes, one of them +inf: dense pulls
    of short lists.  Finite keys are folded by numpy in 64 bits."""
    lists = [[np.inf], [0, np.inf, 1], [np.inf, -3], [-3, np.inf], [-np.inf, np.inf], [-1] * 9 + [np.inf] + [2] * 8,
             [np.inf] + [0] * 19, [-np.inf], [-np.inf, 1], [-np.inf] * 9, [1, 2, 3]]
    mids = 20
    src, dst, w = [], [], []
    for s in range(sources):
        src += [s] * mids
        dst += list(range(200, 200 + mids))
        w += [0.0] * mids
    for t, terms in enumerate(lists):
        src += list(range(200, 200 + len(terms)))
        dst += [300 + t] * len(terms)
        w += terms
    src, dst, w = np.int32(src), np.int32(dst), np.float32(w)
    wl = W.Workload("lse", W.LSE_RULES, {"edge": (("i32", "i32", "f32"), [src, dst, w]),
                                         "source": (("i32",), [np.arange(sources, dtype=np.int32)])},
                    {"score": ("i32", "i32", "f32")})
    print(f"case: one infinite term sources={sources} batched_rounds={batched_rounds}", flush=True)
    rels, stats, _ = engine_run(wl, options={"batched_rounds": batched_rounds, "profile": 1})
    assert stats["pull_launches"] > 0
    s, y, p = rels["score"]
    assert len(s) == sources * (mids + len(lists))
    for t, terms in enumerate(lists):
        got, x = p[y == 300 + t], np.float64(terms)
        m = x.max()
        want = m if np.isinf(m) else m + np.log(np.exp(x - m).sum())
        assert len(got) == sources
        assert np.all(got == want) if np.isinf(m) else np.all(np.abs(got - want) <= LSE_TOL * max(1, abs(want)))


FORMS = {
    "one_add": ("P is P1 + W", {}),
    "two_adds": ("P is P1 + W + 0.0", {}),
    "rounds_one_by_one": ("P is P1 + W", {"batched_rounds": 0}),
    "hashed": ("P is P1 + W", {"index_mode": 1}),
    "hashed_one_by_one": ("P is P1 + W", {"index_mode": 1, "batched_rounds": 0}),
}


@pytest.mark.parametrize("inf", [np.inf, -np.inf])
@pytest.mark.parametrize("sources", [1, 40, 64, 130])
@pytest.mark.parametrize("degree", [3, 40])
@pytest.mark.parametrize("form", list(FORMS))
def test_infinite_log_weights(form, degree, sources, inf):
    """Alone, next to finite values and several in a key, met in one pass and in different passes."""
    layers, width = 4, 50
    rng = np.random.default_rng(degree + sources)
    src = np.repeat(np.arange((layers - 1) * width), degree)
    ahead = np.where(src // width + 2 < layers, 1 + (rng.random(src.size) < 0.2), 1)  # some skip a layer
    dst = (src // width + ahead) * width + rng.integers(0, width, src.size)
    e = np.unique(np.stack([src, dst], 1), axis=0).astype(np.int32)
    w = -rng.random(len(e)).astype(np.float32)
    if inf > 0:
        w[rng.random(len(e)) < (0.05 if degree == 3 else 0.01)] = inf
    else:  # every way into some nodes
        w[(e[:, 1] % 7 == 0) | (rng.random(len(e)) < 0.05)] = inf
    expr, opts = FORMS[form]
    rules = f"score(S,Y,logsumexp(P)) :- source(S), edge(S,Y,P).\nscore(S,Y,logsumexp(P)) :- score(S,Z,P1), edge(Z,Y,W), {expr}.\n"
    wl = W.Workload("lse", rules, {"edge": (("i32", "i32", "f32"), [e[:, 0].copy(), e[:, 1].copy(), w]),
                                   "source": (("i32",), [np.arange(sources, dtype=np.int32)])},
                    {"score": ("i32", "i32", "f32")})
    print(f"case: infinite weights {form} degree={degree} sources={sources} inf={inf}", flush=True)
    ref = evaluate(wl.rules, wl.edb, wl.idb).relations["score"][1]
    got = engine_run(wl, options=opts)[0]["score"]
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    special = ~np.isfinite(ref[2])
    assert special.any() and not np.isnan(ref[2]).any()
    assert np.array_equal(got[2][special], ref[2][special])
    g, r = got[2][~special].astype(np.float64), ref[2][~special].astype(np.float64)
    assert np.all(np.abs(g - r) <= LSE_TOL * np.maximum(1, np.abs(r)))


@pytest.mark.parametrize("index_mode", [0, 1])
def test_infinite_groups(index_mode):
    from paper_2609_27203_amd import xlh
    v = np.float32([np.inf, 0, 1, -np.inf, -np.inf, -np.inf, np.inf, np.inf, 3, np.inf, -np.inf, 2, 0, 0, -np.inf])
    x = np.repeat(np.arange(5, dtype=np.int32), 3)
    print(f"case: infinite groups index_mode={index_mode}", flush=True)
    ctx = xlh.Context(device=0, workspace_bytes=256 << 20)
    ctx.set_option("index_mode", index_mode)
    ctx.relation("e", ("i32", "i32", "f32")).load([x, np.tile(np.arange(3, dtype=np.int32), 5), v])
    ctx.relation("s", ("i32", "f32"))
    ctx.compile("s(X,logsumexp(V)) :- e(X,_,V).").run()
    got = ctx.relations["s"].read()[1]
    assert np.array_equal(got[:4], np.float32([np.inf, -np.inf, np.inf, np.inf])) and abs(got[4] - np.log(2)) < 1e-6
    ctx.close()
