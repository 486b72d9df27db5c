"""First hash tables of recursive set heads: no larger than the rows ask for, widened where a head fills."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

I2 = ("i32", "i32")
REACH = """
reach(S,Y) :- source(S), edge(S,Y).
reach(S,Y) :- reach(S,Z), edge(Z,Y).
"""


def _sparse_ids(n, rng):
    return np.unique(rng.integers(0, 2**31 - 1, n + n // 8 + 64))[:n].astype(np.int32)


def _reach(src, dst, n, sources):
    """(source, node) pairs by breadth-first search over nodes 0..n-1."""
    order = np.argsort(src, kind="stable")
    dst = dst[order]
    off = np.searchsorted(src[order], np.arange(n + 1))
    rows = []
    for s in sources:
        seen = np.zeros(n, bool)
        front = np.array([s])
        while len(front):
            nxt = np.unique(np.concatenate([dst[off[v]:off[v + 1]] for v in front] or [front[:0]]))
            front = nxt[~seen[nxt]]
            seen[front] = True
        hit = np.flatnonzero(seen)
        rows.append(np.c_[np.full(len(hit), s), hit])
    return np.concatenate(rows)


def _run(edge, source, workspace, log2):
    from paper_2609_27203_amd import xlh
    ctx = xlh.Context(device=0, workspace_bytes=workspace)
    ctx.set_option("hash_min_log2", log2)
    ctx.relation("edge", I2).load(edge)
    ctx.relation("source", ("i32",)).load([source])
    ctx.relation("reach", I2)
    stats = ctx.compile(REACH).run()
    rows = np.stack(ctx.relations["reach"].read(), 1)
    ctx.close()
    return rows, stats


def test_few_rows_from_many_edges():
    # 5 M edges among other nodes; two sources on a chain of 20.  Eight slots a
    # joined row would be 2^26 slots of 16 bytes (with the row list), a GiB.
    print("case: first table, few rows from many edges", flush=True)
    rng = np.random.default_rng(5)
    m = 5_000_000
    ids = _sparse_ids(1_250_000, rng)
    src, dst = 100 + rng.integers(0, len(ids) - 100, m), 100 + rng.integers(0, len(ids) - 100, m)
    edge = [np.r_[ids[src], ids[:20]], np.r_[ids[dst], ids[1:21]]]
    rows, stats = _run(edge, ids[:2], 40 << 30, 22)
    want = [(s, y) for s in (0, 1) for y in range(s + 1, 21)]
    assert np.array_equal(rows, np.array([(ids[s], ids[y]) for s, y in want]))
    assert stats["table_grows"] == 0
    assert stats["peak_workspace_bytes"] < 1 << 30  # edges, their index and its build, 2^25 slots


@pytest.mark.parametrize("n,m,log2", [(60_000, 400_000, 18), (60_000, 400_000, 19), (30_000, 100_000, 18)])
def test_head_that_fills(n, m, log2):
    print(f"case: first table, head that fills n={n} m={m} log2={log2}", flush=True)
    rng = np.random.default_rng(n + log2)
    ids = _sparse_ids(n, rng)
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    rows, stats = _run([ids[src], ids[dst]], ids[:40], 4 << 30, log2)
    want = _reach(src, dst, n, range(40))
    assert np.array_equal(rows, np.c_[ids[want[:, 0]], ids[want[:, 1]]])
    assert log2 != 18 or stats["table_grows"] > 0
