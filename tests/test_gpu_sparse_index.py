"""Compacted join indexes searched through buckets of the key's high bits, and
negation tables kept as bitmaps or as keys that need no sort: every distribution
of keys that changes the form, against Python sets."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

I2 = ("i32", "i32")


def _keys(kind, n, rng):
    if kind == "uniform":
        return rng.integers(-2**31, 2**31, n)
    if kind == "extremes":
        return np.r_[-2**31, 2**31 - 1, rng.integers(-2**31, 2**31, n)]
    if kind == "cluster":  # one bucket holds nearly every key
        return np.r_[2**31 - 1, -2**31 + rng.integers(0, 5000, n)]
    if kind == "two_clusters":
        return np.r_[rng.integers(0, 300, n), 2**30 + 2**22 + rng.integers(0, 300, n)]
    return np.r_[7, 7 + 2**27]  # two distinct keys


@pytest.mark.parametrize("n", [1, 60, 5000, 40_000])
@pytest.mark.parametrize("kind", ["uniform", "extremes", "cluster", "two_clusters", "pair"])
def test_join_over_sparse_keys(kind, n):
    from paper_2609_27203_amd import xlh
    print(f"case: sparse join {kind} n={n}", flush=True)
    rng = np.random.default_rng(n)
    keys = _keys(kind, n, rng).astype(np.int32)
    probes = np.r_[keys, np.int32([-2**31, 2**31 - 1, 0, 6, 8]), rng.integers(-2**31, 2**31, 50)].astype(np.int32)
    a = [np.arange(len(probes), dtype=np.int32), probes]
    b = [keys, rng.integers(0, 1000, len(keys)).astype(np.int32)]
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    ctx.relation("a", I2).load(a)
    ctx.relation("b", I2).load(b)
    ctx.relation("j", I2)
    ctx.compile("j(X,Z) :- a(X,Y), b(Y,Z).").run()
    by = {}
    for k, z in set(zip(b[0].tolist(), b[1].tolist())):
        by.setdefault(k, []).append(z)
    want = sorted({(x, z) for x, y in zip(*[c.tolist() for c in a]) for z in by.get(y, ())})
    assert list(zip(*[c.tolist() for c in ctx.relations["j"].read()])) == want
    ctx.close()


NEG = """
keep(X) :- e(X,_), not one(X).
pairs(X,Y) :- e(X,Y), not two(X,Y).
turned(X,Y) :- e(X,Y), not two(Y,X).
lone(X,Y) :- e(X,Y), not two(_,Y).
fixed(X,Y) :- e(X,Y), not two(X,3).
derived(X,Y) :- e(X,Y), not gone(Y,X).
gone(Y,X) :- two(X,Y).
"""


@pytest.mark.parametrize("span,lo", [(50, 0), (50, -25), (100_000, 0), (100_000, -50_000), (2**31 - 1, 0),
                                     (2**32 - 1, -2**31)])
def test_negated_relations(span, lo):
    from paper_2609_27203_amd import xlh
    print(f"case: negation span={span} lo={lo}", flush=True)
    rng = np.random.default_rng(span % 1000)
    n = 3000
    draw = lambda m: (lo + rng.integers(0, min(span, 2**31 - 1), m) * max(1, span // (2**31 - 1))).astype(np.int32)  # noqa: E731
    x, y = draw(n), draw(n)
    tx, ty = np.r_[x[: n // 3], draw(400)], np.r_[y[: n // 3], draw(400)]
    tx[:5], ty[:5] = x[:5], 3
    one = np.r_[x[: n // 2], draw(100)]
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    ctx.set_option("hash_min_log2", 16)
    for name, cols in (("e", [x, y]), ("two", [tx, ty]), ("one", [one])):
        ctx.relation(name, ("i32",) * len(cols)).load(cols)
    idb = {"keep": 1, "pairs": 2, "turned": 2, "lone": 2, "fixed": 2, "derived": 2, "gone": 2}
    for name, k in idb.items():
        ctx.relation(name, ("i32",) * k)
    ctx.compile(NEG).run()
    e, two = set(zip(x.tolist(), y.tolist())), set(zip(tx.tolist(), ty.tolist()))
    ones, seconds = set(one.tolist()), {b for _, b in two}
    want = {"keep": {(a,) for a, _ in e if a not in ones}, "pairs": e - two,
            "turned": {(a, b) for a, b in e if (b, a) not in two}, "lone": {(a, b) for a, b in e if b not in seconds},
            "fixed": {(a, b) for a, b in e if (a, 3) not in two}, "derived": e - two,
            "gone": {(b, a) for a, b in two}}
    for name, rows in want.items():
        assert list(zip(*[c.tolist() for c in ctx.relations[name].read()])) == sorted(rows), name
    ctx.close()


@pytest.mark.parametrize("low,high", [(-2**31, 2**31 - 1), (-2**31, 2**31 - 2), (-2**31 + 1, 2**31 - 1)])
def test_negated_column_over_the_whole_range(low, high):
    """2^25 rows whose bounds are (nearly) those of int32: a bitmap of up to 2^32 bits."""
    import torch

    from paper_2609_27203_amd import xlh
    print(f"case: negation over [{low}, {high}]", flush=True)
    n = 1 << 25
    q = low + 128 * torch.arange(n, dtype=torch.int64, device="cuda")
    q[-1] = high
    rng = np.random.default_rng(7)
    x = np.r_[-2**31, 2**31 - 1, high, low, low + 1, high - 1, low + 128 * rng.integers(0, n - 1, 500),
              rng.integers(-2**31, 2**31, 500)].astype(np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=4 << 30)
    ctx.relation("q", ("i32",)).load([q.to(torch.int32)])
    ctx.relation("e", ("i32",)).load([x])
    ctx.relation("keep", ("i32",))
    ctx.compile("keep(X) :- e(X), not q(X).").run()
    off = x.astype(np.int64) - low
    in_q = (x == high) | ((off >= 0) & (off % 128 == 0) & (off // 128 < n - 1))
    assert 0 < in_q.sum() < len(x)
    assert np.array_equal(ctx.relations["keep"].read()[0], np.unique(x[~in_q]))
    ctx.close()
