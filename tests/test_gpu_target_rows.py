"""Rows of target-major sum heads written rank by rank: source and target
counts around the 32-rank and 64-target steps, one and several steps per tile,
with and without absent slots.  Path counts are integers: compared exactly
with the hash-table form, and the readout must ascend strictly."""
import numpy as np
import pytest

from helpers import engine_run
from paper_2609_27203_amd import workloads as W

pytestmark = pytest.mark.gpu

RULES = """
npaths(S,Y,sum(C)) :- source(S), C is 1, edge(S,Y,_).
npaths(S,Y,sum(C)) :- npaths(S,Z,C1), edge(Z,Y,_), C is C1.
"""


@pytest.mark.parametrize("layers,width,degree,sources", [
    (3, 2, 1, 1), (3, 7, 2, 2), (4, 16, 2, 16), (3, 21, 1, 21), (2, 32, 3, 31), (3, 32, 2, 32), (4, 33, 3, 33),
    (5, 51, 2, 50), (3, 86, 4, 64), (3, 90, 1, 65), (6, 100, 3, 96), (4, 500, 2, 97), (12, 2600, 2, 280)])
def test_rows_match_the_hashed_form(layers, width, degree, sources):
    wl = W.layered_dag(layers, width, degree, sources, seed=layers * width)
    wl = W.Workload("npaths", RULES, wl.edb, {"npaths": ("i32", "i32", "i32")})
    print(f"case: target rows {layers} x {width} degree {degree} sources {sources}", flush=True)
    rels, stats, _ = engine_run(wl, workspace_bytes=2 << 30)
    hashed, hstats, _ = engine_run(wl, workspace_bytes=2 << 30, options={"index_mode": 1})
    s, y, _ = rels["npaths"]
    assert stats["derived_tuples"] == hstats["derived_tuples"] == len(s) > 0
    key = (s.astype(np.int64) << 32) | y.astype(np.int64)
    assert np.all(key[1:] > key[:-1])
    for g, w in zip(rels["npaths"], hashed["npaths"]):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("width,degree,sources", [(1, 1, 1), (33, 33, 40), (70, 70, 65), (300, 41, 7), (700, 3, 100)])
def test_pulled_marks_match_a_host_sum(width, degree, sources):
    """logsumexp rounds that pull straight from the mark words: in-degrees past
    a step of 32, words with few marks (queued) and full ones, targets across
    words.  A layer's fold of n terms in 32 bits is off by at most n + 8
    roundings (exp, log and rescale counted as eight), and the carried value
    by one of its own per layer."""
    rng = np.random.default_rng(width * degree)
    layers, degree = 3, min(degree, width)
    to = np.stack([rng.choice(width, size=degree, replace=False) for _ in range(layers * width)])
    src = np.repeat(np.arange(layers * width), degree)
    dst = to.reshape(-1) + (src // width + 1) * width
    w = -rng.random(src.size).astype(np.float32)
    srcs = np.sort(rng.choice(layers * width, size=sources % width + 1, replace=False)).astype(np.int32)
    wl = W.Workload("lse", W.LSE_RULES, {
        "edge": (("i32", "i32", "f32"), [src.astype(np.int32), dst.astype(np.int32), w]),
        "source": (("i32",), [srcs])}, {"score": ("i32", "i32", "f32")})
    print(f"case: pulled marks width {width} degree {degree} sources {len(srcs)}", flush=True)
    rels, _, _ = engine_run(wl, workspace_bytes=2 << 30)
    total = np.zeros((len(srcs), (layers + 1) * width))  # sums of path products
    prod = np.exp(w.astype(np.float64))
    for i, s in enumerate(srcs):
        total[i, s] = 1.0
        for l in range(s // width, layers):
            e = slice(l * width * degree, (l + 1) * width * degree)
            np.add.at(total[i], dst[e], total[i, src[e]] * prod[e])
        total[i, s] = 0.0
    at, y = np.nonzero(total)
    want = np.log(total[at, y])
    got = rels["score"]
    assert np.array_equal(got[0], srcs[at]) and np.array_equal(got[1], y)
    bound = layers * (degree + 8 + np.abs(want).max()) * 2.0**-24
    assert np.abs(got[2] - want).max() <= bound
