"""Gathered rounds, h(X,Y) :- e1(X,A), h(A,B), e2(Y,B): the unions applied per
head row against the pairwise join (gather_rounds 0) and the oracle, all
exact.  Lists of A values around the four taken at a time and the 16 beyond which
the unions are ORed by atomics; bitmaps on both sides of the 8 MB from which a
round is two launches, rows around a lane group's 32 and 128 words and a
wavefront's 64, delta words with few and with more than 512 bits."""
import numpy as np
import pytest

from helpers import engine_run
from oracle import evaluate
from paper_2609_27203_amd import workloads as W

pytestmark = pytest.mark.gpu

RULES = """
sg(X,Y) :- flat(X,Y).
sg(X,Y) :- up(X,A), sg(A,B), up(Y,B).
"""
T = ("i32", "i32")


def _graph(n, width, fan, seed):
    """Ids spread over n; a hub child with `fan` parents, others with up to three, four generations."""
    rng = np.random.default_rng(seed)
    ids = np.unique(np.r_[0, n - 1, rng.choice(n, min(n, 4 * width), replace=False)]).astype(np.int32)
    rng.shuffle(ids)
    gens = np.array_split(ids, 4)
    up = []
    for parents, children in zip(gens, gens[1:]):
        for j, c in enumerate(children):
            k = min(fan if j == 0 else rng.integers(1, 4), len(parents))
            up += [(c, p) for p in rng.choice(parents, k, replace=False)]
    a, b = rng.choice(gens[0], 3 * width), rng.choice(gens[0], 3 * width)
    up = np.array(up, np.int32)
    return {"flat": (T, [a, b]), "up": (T, [up[:, 0].copy(), up[:, 1].copy()])}


@pytest.mark.parametrize("n,width,fan", [
    (40, 8, 1), (400, 30, 4), (2048, 90, 16), (2300, 120, 100), (8192, 60, 16), (8193, 60, 16), (8300, 30, 1),
    (8300, 40, 4), (9000, 40, 5), (10240, 40, 8), (10241, 60, 15), (12288, 90, 16), (12289, 90, 17), (16385, 70, 16),
    (9000, 100, 13), (9000, 100, 80)])
@pytest.mark.parametrize("batch", [0, 4])
def test_lists_and_widths(n, width, fan, batch):
    wl = W.Workload("sg", RULES, _graph(n, width, fan, n + fan), {"sg": T})
    if n in (2048, 12288):  # a first generation that is related throughout: full delta words
        a = np.unique(wl.edb["flat"][1][0])
        wl.edb["flat"] = (T, [np.repeat(a, n), np.tile(np.arange(n, dtype=np.int32), len(a))])
    print(f"case: gathered n={n} width={width} fan={fan} batch={batch}", flush=True)
    rels, stats, _ = engine_run(wl, options={"batched_rounds": batch, "profile": 1})
    assert stats["gather_launches"] > 0
    ref = evaluate(wl.rules, wl.edb, wl.idb)
    for g, w in zip(rels["sg"], ref.relations["sg"][1]):
        assert np.array_equal(g, w)
    pairs, pstats, _ = engine_run(wl, options={"batched_rounds": batch, "gather_rounds": 0})
    for g, w in zip(rels["sg"], pairs["sg"]):
        assert np.array_equal(g, w)
    for key in ("delta_rows", "iterations", "new_tuples_total", "derived_tuples"):
        assert stats[key] == pstats[key], key
