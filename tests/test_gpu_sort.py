"""The radix sort through the public entry points: loads (sort and
deduplication), reads of unsorted relations and index builds, at the sizes
where its forms change (one workgroup in LDS, the scatter that reads the whole
count table, the scanned table, several tiles per workgroup) and with skewed,
constant and full-range keys.  Compared bit for bit with numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [4095, 4096, 4097, 5000, 65535, 65536, 65537, 70001, 1 << 20, (1 << 20) + 1, (1 << 22) - 1, (1 << 22) + 5,
         5_300_011]


def _cols(kind, n, rng):
    if kind == "full":
        return [rng.integers(-2**31, 2**31, n).astype(np.int32), rng.integers(-2**31, 2**31, n).astype(np.int32)]
    if kind == "narrow":
        return [rng.integers(-5, 900, n).astype(np.int32), rng.integers(0, 700, n).astype(np.int32)]
    if kind == "constant":
        return [np.full(n, 7, np.int32), rng.integers(0, 3, n).astype(np.int32)]
    if kind == "skewed":  # most rows in a few keys
        a = np.minimum(rng.geometric(0.3, n), 2**20).astype(np.int32)
        return [a, rng.zipf(1.3, n).clip(0, 2**24).astype(np.int32)]
    a = np.sort(rng.integers(0, 2**26, n)).astype(np.int32)  # already in order
    return [a, a[::-1].copy()]


def _canonical(cols):
    order = np.lexsort(cols[::-1])
    cols = [c[order] for c in cols]
    keep = np.ones(len(order), bool)
    keep[1:] = np.any([c[1:] != c[:-1] for c in cols], axis=0)
    return [c[keep] for c in cols]


@pytest.mark.parametrize("kind", ["full", "narrow", "constant", "skewed", "ordered"])
@pytest.mark.parametrize("n", SIZES)
def test_load_sorts_and_deduplicates(kind, n):
    import torch

    from paper_2609_27203_amd import xlh
    print(f"case: load {kind} n={n}", flush=True)
    cols = _cols(kind, n, np.random.default_rng(n))
    want = _canonical(cols)
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    rel = ctx.relation("r", ("i32", "i32"))
    rel.load([torch.from_numpy(c).cuda() for c in cols])
    for g, w in zip(rel.read_device(), want):
        assert np.array_equal(g.cpu().numpy(), w)
    ctx.close()


@pytest.mark.parametrize("n", [3000, 9000, 66000, 300_000])
def test_index_by_second_column_and_hashed_readout(n):
    """rev(Y,X) over a hash-table head: index builds and the unsorted readout."""
    from paper_2609_27203_amd import xlh
    print(f"case: index and unsorted readout n={n}", flush=True)
    rng = np.random.default_rng(n)
    x, y = rng.integers(-2**30, 2**30, n).astype(np.int32), rng.integers(0, n // 2, n).astype(np.int32)
    ctx = xlh.Context(device=0, workspace_bytes=1 << 30)
    ctx.set_option("index_mode", 1)
    ctx.relation("r", ("i32", "i32")).load([x, y])
    ctx.relation("k", ("i32",)).load([np.arange(n // 2, dtype=np.int32)])
    ctx.relation("rev", ("i32", "i32"))
    ctx.compile("rev(Y,X) :- k(Y), r(X,Y).").run()
    for g, w in zip(ctx.relations["rev"].read(), _canonical([y, x])):
        assert np.array_equal(g, w)
    ctx.close()
