"""Grouped aggregates of non-recursive rules: groups that span lanes, wavefronts
and single rows, in driver order and shuffled by a join, one and two key
columns, dense and hashed heads, against numpy in the engine's arithmetic."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RULES = """
low(X,min(V)) :- e(X,Y,V).
high(X,max(V)) :- e(X,Y,V).
n(X,count(Y)) :- e(X,Y,_).
total(X,sum(K)) :- f(X,Y,K).
bylow(Y,min(V)) :- e(_,Y,V).
pairhigh(X,Y,max(V)) :- e(X,Y,V).
pairtotal(Y,X,sum(K)) :- f(X,Y,K).
two(X,min(D)) :- e(X,Y,V), e(Y,_,U), D is V + U.
"""
F, I = ("i32", "f32"), ("i32", "i32")
IDB = {"low": F, "high": F, "n": I, "total": I, "bylow": F, "pairhigh": ("i32", "i32", "f32"),
       "pairtotal": ("i32", "i32", "i32"), "two": F}


def _fold(keys, v, how):
    order = np.lexsort(keys[::-1])
    keys, v = [k[order] for k in keys], v[order]
    start = np.ones(len(v), bool)
    start[1:] = np.any([k[1:] != k[:-1] for k in keys], axis=0)
    at = np.flatnonzero(start)
    return [k[at] for k in keys] + [how.reduceat(v, at)]


@pytest.mark.parametrize("index_mode", [0, 1])
@pytest.mark.parametrize("shape", ["single_rows", "pairs", "tens", "waves", "hub", "negative"])
def test_grouped_folds(shape, index_mode):
    from paper_2609_27203_amd import xlh
    print(f"case: groups {shape} index_mode={index_mode}", flush=True)
    rng = np.random.default_rng(len(shape))
    n = 6000
    groups = {"single_rows": n, "pairs": n // 2, "tens": n // 10, "waves": 40, "hub": 3, "negative": 500}[shape]
    x = rng.permutation(n) if shape == "single_rows" else rng.integers(0, groups, n)
    y = rng.integers(0, groups, n)
    if shape == "negative":
        x, y = x - 250, y - 100
    xy = np.unique(np.stack([x, y], 1), axis=0).astype(np.int32)
    x, y = xy[:, 0].copy(), xy[:, 1].copy()
    v = (rng.standard_normal(len(x)) * 10).astype(np.float32)
    k = rng.integers(-1000, 1000, len(x)).astype(np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    ctx.set_option("index_mode", index_mode)
    ctx.relation("e", ("i32", "i32", "f32")).load([x, y, v])
    ctx.relation("f", ("i32", "i32", "i32")).load([x, y, k])
    for name, types in IDB.items():
        ctx.relation(name, types)
    ctx.compile(RULES).run()
    lows = dict(zip(*[c.tolist() for c in _fold([x], v, np.minimum)]))
    near = np.array([lows.get(int(b), np.inf) for b in y], np.float32)
    ok = np.isfinite(near)
    want = {"low": _fold([x], v, np.minimum), "high": _fold([x], v, np.maximum),
            "n": _fold([x], np.ones(len(x), np.int32), np.add), "total": _fold([x], k, np.add),
            "bylow": _fold([y], v, np.minimum), "pairhigh": _fold([x, y], v, np.maximum),
            "pairtotal": _fold([y, x], k, np.add), "two": _fold([x[ok]], (v + near)[ok], np.minimum)}
    for name, cols in want.items():
        got = ctx.relations[name].read()
        assert len(got[0]) == len(cols[0]), name
        for g, w in zip(got, cols):
            assert np.array_equal(g, w.astype(g.dtype)), name
    ctx.close()


@pytest.mark.parametrize("index_mode", [0, 1])
def test_min_of_extreme_values(index_mode):
    """Infinities and the largest finite values, alone and next to others in their group."""
    from paper_2609_27203_amd import xlh
    print(f"case: extreme values index_mode={index_mode}", flush=True)
    big = np.finfo(np.float32).max
    x = np.repeat(np.arange(6, dtype=np.int32), 3)
    y = np.tile(np.arange(3, dtype=np.int32), 6)
    v = np.float32([np.inf] * 3 + [-np.inf] * 3 + [big, np.inf, -big] + [-np.inf, np.inf, 0] + [0.0, 1e-45, -1e-45]
                   + [np.inf, big, big])
    ctx = xlh.Context(device=0, workspace_bytes=256 << 20)
    ctx.set_option("index_mode", index_mode)
    ctx.relation("e", ("i32", "i32", "f32")).load([x, y, v])
    ctx.relation("low", F)
    ctx.relation("high", F)
    ctx.compile("low(X,min(V)) :- e(X,Y,V).\nhigh(X,max(V)) :- e(X,Y,V).").run()
    assert np.array_equal(ctx.relations["low"].read()[1], v.reshape(6, 3).min(1))
    assert np.array_equal(ctx.relations["high"].read()[1], v.reshape(6, 3).max(1))
    ctx.close()


SCAN_RULES = """
same(X,Y) :- e(X,Y).
turned(Y,X) :- e(X,Y).
either(X,Y) :- e(X,Y).
either(X,Y) :- e(Y,X), X != 7.
first(X) :- e(X,_).
second(Y) :- e(_,Y), not first(Y).
none(X,Y) :- e(X,Y), X < -5.
joined(X,Z) :- same(X,Y), turned(Y,Z), X != Z.
"""


@pytest.mark.parametrize("index_mode", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 2047, 2049, 70_000])
@pytest.mark.parametrize("span", [2**17, 2**31 - 8])
def test_scanned_sets_over_wide_domains(n, span, index_mode):
    """Set heads of scans whose bitmap would be far larger than their rows (sorted
    candidate keys of 32 and 64 bits), and rules that join them afterwards."""
    from paper_2609_27203_amd import xlh
    print(f"case: scanned sets n={n} span={span} index_mode={index_mode}", flush=True)
    rng = np.random.default_rng(n)
    x = np.r_[0, span, rng.integers(0, span, n)].astype(np.int32)
    y = np.r_[span, 5, rng.integers(0, span, n)].astype(np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    ctx.set_option("index_mode", index_mode)
    ctx.set_option("hash_min_log2", 18)
    ctx.relation("e", I).load([x, y])
    two = ("same", "turned", "either", "none", "joined")
    for name in two:
        ctx.relation(name, I)
    for name in ("first", "second"):
        ctx.relation(name, ("i32",))
    stats = ctx.compile(SCAN_RULES).run()
    e = set(zip(x.tolist(), y.tolist()))
    back = {}
    for a, b in e:
        back.setdefault(b, []).append(a)
    firsts = {a for a, _ in e}
    want = {"same": e, "turned": {(b, a) for a, b in e}, "none": set(),
            "either": e | {(b, a) for a, b in e if b != 7},
            "joined": {(a, c) for a, b in e for c in back[b] if a != c},
            "first": {(a,) for a in firsts}, "second": {(b,) for _, b in e if b not in firsts}}
    for name, rows in want.items():
        got = ctx.relations[name].read()
        assert list(zip(*[c.tolist() for c in got])) == sorted(rows), name
    assert stats["derived_tuples"] == sum(len(r) for r in want.values())
    ctx.close()


def test_scanned_set_capacity_and_resume():
    """max_rows bounds the distinct rows; a relation with rows keeps them."""
    from paper_2609_27203_amd import xlh
    print("case: scanned set capacity and resume", flush=True)
    x = np.arange(1000, dtype=np.int32) * 1_000_003 % 2**30
    for limit, ok in ((1000, True), (999, False)):
        ctx = xlh.Context(device=0, workspace_bytes=256 << 20)
        ctx.relation("e", I).load([np.r_[x, x], np.r_[x, x]])
        ctx.relation("f", I).load([np.r_[x, x], np.r_[x[::-1], x]])
        out = ctx.relation("out", I, max_rows=limit)
        prog = ctx.compile("out(X,Y) :- e(X,Y).\nout(Y,X) :- e(X,Y).")
        if not ok:
            with pytest.raises(xlh.XlError) as ei:
                prog.run()
            assert ei.value.status_name == "XL_CAPACITY_EXCEEDED"
            continue
        prog.run()
        assert out.size() == 1000
        out.load([np.int32([3]), np.int32([4])])
        ctx.relation("more", I)
        with pytest.raises(xlh.XlError):  # 1,001 rows now
            prog.run()
        ctx.close()


RECEIPT_RULES = """
tc(X,Y) :- e(X,Y).
tc(X,Y) :- tc(X,Z), e(Z,Y).
far(X,max(Y)) :- tc(X,Y).
near(X,min(Y)) :- tc(X,Y).
n(X,count(Y)) :- tc(X,Y).
total(X,sum(Y)) :- tc(X,Y).
wide(X,Y) :- w(X,Y).
"""


@pytest.mark.parametrize("profile", [0, 1])
@pytest.mark.parametrize("passes", [3, 255, 256, 300])
def test_receipt_after_many_passes(passes, profile):
    """Strata after the last recorded round still count in new_tuples_total."""
    from paper_2609_27203_amd import xlh
    print(f"case: receipt passes={passes} profile={profile}", flush=True)
    x = np.arange(passes, dtype=np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=256 << 20)
    ctx.set_option("profile", profile)
    ctx.relation("e", ("i32", "i32")).load([x, x + 1])
    ctx.relation("w", ("i32", "i32")).load([x * 7_000_003, x * 5_000_011])
    for name, k in (("tc", 2), ("far", 2), ("near", 2), ("n", 2), ("total", 2), ("wide", 2)):
        ctx.relation(name, ("i32",) * k)
    st = ctx.compile(RECEIPT_RULES).run()
    assert st["rounds_recorded"] >= passes + 5
    assert st["derived_tuples"] == passes * (passes + 1) // 2 + 5 * passes
    assert st["new_tuples_total"] == st["derived_tuples"]
    if st["rounds_recorded"] <= 256:
        assert sum(st["delta_rows"]) == st["derived_tuples"]
    ctx.close()


PROJECTED_RULES = """
lead(X,Y) :- e(X,Y,_).
turned(Y,X) :- e(X,Y,_).
both(X,Y) :- e(X,Y,_).
both(Y,X) :- e(X,Y,_).
fixed(Y,X) :- e(X,Y,5).
twice(Z,X) :- e(X,X,Z).
outer(Z,X) :- e(X,_,Z).
"""


@pytest.mark.parametrize("workspace", [64, 1024])
@pytest.mark.parametrize("n", [1, 2049, 200_000])
def test_scanned_sets_of_wider_drivers(n, workspace):
    """Heads that drop a driver column (candidates repeat), fix one by a constant or
    by another column, or keep rows in order, with much and little room."""
    from paper_2609_27203_amd import xlh
    print(f"case: sets of wider drivers n={n} workspace={workspace} MB", flush=True)
    rng = np.random.default_rng(n)
    a = np.r_[0, 2**31 - 2, rng.integers(0, 2**31 - 1, 40)].astype(np.int32)
    x, y = a[rng.integers(0, len(a), (2, n))]
    x[0], y[0] = 0, 2**31 - 2
    z = rng.integers(0, 9, n).astype(np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=workspace << 20)
    ctx.set_option("hash_min_log2", 12)
    ctx.relation("e", ("i32", "i32", "i32")).load([x, y, z])
    e = set(zip(x.tolist(), y.tolist(), z.tolist()))
    want = {"lead": {(p, q) for p, q, _ in e}, "turned": {(q, p) for p, q, _ in e},
            "both": {r for p, q, _ in e for r in ((p, q), (q, p))}, "fixed": {(q, p) for p, q, r in e if r == 5},
            "twice": {(r, p) for p, q, r in e if p == q}, "outer": {(r, p) for p, _, r in e}}
    for name in want:
        ctx.relation(name, I)
    stats = ctx.compile(PROJECTED_RULES).run()
    for name, rows in want.items():
        assert list(zip(*[c.tolist() for c in ctx.relations[name].read()])) == sorted(rows), name
    assert stats["derived_tuples"] == stats["new_tuples_total"] == sum(len(r) for r in want.values())
    ctx.close()
