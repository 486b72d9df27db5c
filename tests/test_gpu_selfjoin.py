"""Self-joined closure, path(X,Y) :- path(X,Z), path(Z,Y), over a dense head:
rounds that OR whole bitmap rows against the generic join of each pair
(batched_rounds 0), the hash-table form and the oracle: rows, per-pass deltas,
pass counts and candidate counts, all exact."""
import numpy as np
import pytest

from helpers import engine_run
from oracle import evaluate
from paper_2609_27203_amd import workloads as W

pytestmark = pytest.mark.gpu

RULES = """
path(X,Y) :- edge(X,Y).
path(X,Y) :- path(X,Z), path(Z,Y).
"""
SWAPPED = """
path(X,Y) :- edge(X,Y).
path(A,B) :- path(C,B), path(A,C).
"""
IDB = {"path": ("i32", "i32")}


def _graph(nodes, edges, span, shift, seed):
    """Edges over `nodes` ids spread over [shift, shift + span), the extremes among them."""
    rng = np.random.default_rng(seed)
    ids = np.unique(np.r_[0, span - 1, rng.choice(span, min(nodes, span), replace=False)]).astype(np.int32) + shift
    a, b = ids[rng.integers(0, len(ids), edges)], ids[rng.integers(0, len(ids), edges)]
    return {"edge": (("i32", "i32"), [np.r_[a, ids[0], ids[-1]].astype(np.int32),
                                      np.r_[b, ids[-1], ids[0]].astype(np.int32)])}


def _same(got, want):
    for g, w in zip(got["path"], want["path"]):
        assert np.array_equal(g, w)


# row words 1, 2, 16/17, 32/33, 64/65, 128/129, 192/193, 256/257, 384/385, 512 and one above the form's limit
SPANS = [31, 70, 96, 128, 129, 40, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 6144, 6145, 8192, 8193, 12288, 12289, 16384, 16385]


@pytest.mark.parametrize("span", SPANS)
@pytest.mark.parametrize("shift", [0, -700])
def test_row_widths(span, shift):
    edb = _graph(40, 70, span, shift, span)
    wl = W.Workload("sj", RULES, edb, IDB)
    print(f"case: self-join widths span={span} shift={shift}", flush=True)
    ref = evaluate(wl.rules, wl.edb, wl.idb)
    want = {"path": ref.relations["path"][1]}
    rels, stats, _ = engine_run(wl)
    _same(rels, want)
    sizes = ref.sizes["path"]
    assert stats["delta_rows"] == [sizes[0]] + [b - a for a, b in zip(sizes, sizes[1:])]
    generic, gstats, _ = engine_run(wl, options={"batched_rounds": 0})
    _same(generic, want)
    for key in ("delta_rows", "iterations", "candidates_total", "new_tuples_total", "derived_tuples"):
        assert stats[key] == gstats[key], key


@pytest.mark.parametrize("rules", [RULES, SWAPPED])
@pytest.mark.parametrize("batch", [1, 4, 64])
def test_dense_rows_match_the_generic_join(rules, batch):
    """Several listing steps per row (more than 64 words), dense rows, atoms in either order."""
    src, dst = W.uniform_graph(2500, 6000, 3)
    wl = W.Workload("sj_dense", rules, {"edge": (("i32", "i32"), [src, dst])}, IDB)
    print(f"case: self-join dense batch={batch}", flush=True)
    rels, stats, _ = engine_run(wl, options={"batched_rounds": batch})
    generic, gstats, _ = engine_run(wl, options={"batched_rounds": 0})
    hashed, _, _ = engine_run(wl, options={"index_mode": 1})
    linear, _, _ = engine_run(W.Workload("tc", W.TC_RULES, wl.edb, IDB))
    for other in (generic, hashed, linear):
        _same(rels, other)
    for key in ("delta_rows", "iterations", "candidates_total", "new_tuples_total"):
        assert stats[key] == gstats[key], key


def test_column_ranges_apart():
    """First and second columns over different ranges: few Y are also an X."""
    rng = np.random.default_rng(8)
    edb = {"edge": (("i32", "i32"), [rng.integers(0, 300, 900).astype(np.int32),
                                     rng.integers(250, 900, 900).astype(np.int32)])}
    for flip in (False, True):
        cols = edb["edge"][1][::-1] if flip else edb["edge"][1]
        wl = W.Workload("sj_apart", RULES, {"edge": (("i32", "i32"), list(cols))}, IDB)
        print(f"case: self-join ranges apart flip={flip}", flush=True)
        ref = evaluate(wl.rules, wl.edb, wl.idb)
        rels, _, _ = engine_run(wl)
        _same(rels, {"path": ref.relations["path"][1]})


def test_iteration_cap_max_rows_and_resume():
    from paper_2609_27203_amd import xlh
    n = 40
    edb = {"edge": (("i32", "i32"), [np.arange(n, dtype=np.int32), np.arange(1, n + 1, dtype=np.int32)])}
    wl = W.Workload("sj_chain", RULES, edb, IDB)
    print("case: self-join cap, capacity, resume", flush=True)
    rels, stats, ctx = engine_run(wl)
    passes = stats["iterations"]
    for batch in (0, 1, 4):
        for cap in (0, passes - 1):
            with pytest.raises(xlh.XlError) as ei:
                engine_run(wl, max_iterations=cap, options={"batched_rounds": batch})
            assert ei.value.status_name == "XL_CONVERGENCE_FAILURE"
        assert engine_run(wl, max_iterations=passes, options={"batched_rounds": batch})[1]["iterations"] == passes
    small = xlh.Context(device=0, workspace_bytes=64 << 20)
    small.relation("edge", ("i32", "i32")).load(edb["edge"][1])
    small.relation("path", ("i32", "i32"), max_rows=n * (n + 1) // 2 - 1)
    with pytest.raises(xlh.XlError) as ei:
        small.compile(RULES).run()
    assert ei.value.status_name == "XL_CAPACITY_EXCEEDED"
    # a loaded fixpoint plus one new edge: the run resumes from it
    ctx.relations["path"].load(rels["path"])
    ctx.relations["edge"].load([np.r_[edb["edge"][1][0], np.int32(n)], np.r_[edb["edge"][1][1], np.int32(n + 1)]])
    ctx.compile(RULES).run()
    longer, _, _ = engine_run(W.Workload("sj_chain2", RULES, {"edge": (("i32", "i32"), [
        np.arange(n + 1, dtype=np.int32), np.arange(1, n + 2, dtype=np.int32)])}, IDB))
    _same({"path": ctx.relations["path"].read()}, longer)
