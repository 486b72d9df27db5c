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
