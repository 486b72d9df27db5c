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


def _load_and_read(types, cols, device, shift=0, workspace=256 << 20):
    """Load through host or device memory (device columns `shift` bytes past an
    aligned start), read back; returns numpy columns."""
    import ctypes as C

    import torch

    from paper_2609_27203_amd import xlh
    ctx = xlh.Context(device=0, workspace_bytes=workspace)
    rel = ctx.relation("r", types)
    if device:
        keep = []
        for c in cols:
            b = torch.zeros(c.nbytes + 16, dtype=torch.uint8, device="cuda")
            b[shift:shift + c.nbytes] = torch.from_numpy(c.view(np.uint8)).cuda()
            keep.append(b)
        torch.cuda.synchronize()
        ptrs = (C.c_void_p * len(cols))(*[b.data_ptr() + shift for b in keep])
        ctx._check(xlh.lib().xl_relation_load(rel._h, ptrs, len(cols[0]), 1))
        for b, c in zip(keep, cols):  # inputs are only read
            assert np.array_equal(b.cpu().numpy()[shift:shift + c.nbytes], c.view(np.uint8))
    else:
        rel.load(cols)
    out = rel.read()
    ctx.close()
    return out


def _order_images(c):
    if c.dtype == np.float32:
        u = c.view(np.uint32)
        return np.where(u >> 31, ~u, u | np.uint32(1 << 31))
    return c


def _canonical_bits(cols):
    """Canonical rows with float columns in totalOrder, duplicates by bits."""
    img = [_order_images(c) for c in cols]
    order = np.lexsort(img[::-1])
    img = [c[order] for c in img]
    keep = np.ones(len(order), bool)
    keep[1:] = np.any([c[1:] != c[:-1] for c in img], axis=0) if len(order) > 1 else True
    return [c[order][keep] for c in cols]


WIDTHS = {
    # name: (types, column makers); bits of the packed key and what is left of the columns
    "one_column": (("i32",), lambda r, n: [r.integers(-2**31, 2**31, n).astype(np.int32)]),
    "one_float": (("f32",), lambda r, n: [np.r_[np.float32([0.0, -0.0, np.inf, -np.inf]),
                                                r.standard_normal(n).astype(np.float32)]]),
    "constant_columns": (("i32", "i32", "i32"), lambda r, n: [np.full(n, 5, np.int32), np.full(n, -9, np.int32),
                                                              r.integers(0, 50, n).astype(np.int32)]),
    "exactly_32_bits": (("i32", "i32"), lambda r, n: [np.r_[0, 2**16 - 1, r.integers(0, 2**16, n)].astype(np.int32),
                                                      np.r_[0, 2**16 - 1, r.integers(0, 2**16, n)].astype(np.int32)]),
    "exactly_64_bits": (("i32", "f32"), lambda r, n: [np.r_[-2**31, 2**31 - 1, r.integers(-9, 9, n)].astype(np.int32),
                                                      np.r_[np.float32([-np.inf, np.inf]),
                                                            r.standard_normal(n).astype(np.float32)]]),
    "payload": (("i32", "i32", "f32"), lambda r, n: [r.integers(0, 2**20, n).astype(np.int32),
                                                     r.integers(0, 2**14, n).astype(np.int32),
                                                     r.standard_normal(n).astype(np.float32)]),
    "payload_with_runs": (("i32", "i32", "i32"), lambda r, n: [
        np.r_[-2**31, 2**31 - 1, r.integers(0, max(1, n // 40), n)].astype(np.int32),
        np.r_[0, 2**31 - 1, r.integers(0, 2, n)].astype(np.int32), r.integers(-2**31, 2**31, n + 2).astype(np.int32)]),
    "payload_long_run": (("i32", "i32", "f32"), lambda r, n: [
        np.r_[-2**31, 2**31 - 1, np.full(n, 3)].astype(np.int32),
        np.r_[0, 2**31 - 1, np.full(n, 4)].astype(np.int32), r.standard_normal(n + 2).astype(np.float32)]),
    "four_wide_columns": (("i32", "f32", "i32", "f32"), lambda r, n: [
        r.integers(-2**31, 2**31, n).astype(np.int32), r.standard_normal(n).astype(np.float32),
        r.integers(0, 4, n).astype(np.int32), np.float32(r.integers(0, 3, n))]),
    "four_narrow_columns": (("i32", "i32", "i32", "i32"), lambda r, n: [
        r.integers(0, k, n).astype(np.int32) for k in (3, 70, 9, 1000)]),
}


@pytest.mark.parametrize("name", list(WIDTHS))
@pytest.mark.parametrize("n", [2, 47, 60, 4094, 5000, 70001])
def test_load_layouts(name, n):
    types, make = WIDTHS[name]
    cols = make(np.random.default_rng(n), n)
    cols = [np.ascontiguousarray(np.r_[c, c[: len(c) // 3]]) for c in cols]  # a third of the rows twice
    want = _canonical_bits(cols)
    for device, shift in ((False, 0), (True, 0), (True, 4), (True, 2)):
        print(f"case: load layout {name} n={n} device={device} shift={shift}", flush=True)
        for g, w in zip(_load_and_read(types, cols, device, shift), want):
            assert np.array_equal(g.view(np.uint32), w.view(np.uint32))


def test_load_in_a_workspace_that_holds_less():
    """Smaller workspaces down to one that refuses the load: the rows are right or the call is refused."""
    from paper_2609_27203_amd import xlh
    types, make = WIDTHS["payload"]
    n = 50_000
    cols = make(np.random.default_rng(1), n)
    want = _canonical_bits(cols)
    refused = 0
    for ws in [(1 << 20) + i * (1 << 18) for i in range(16)]:
        print(f"case: load in {ws} bytes", flush=True)
        for device in (False, True):
            try:
                got = _load_and_read(types, cols, device, 0, ws)
            except xlh.XlError as e:
                assert e.status_name == "XL_RESOURCE_EXHAUSTED"
                refused += 1
                continue
            for g, w in zip(got, want):
                assert np.array_equal(g.view(np.uint32), w.view(np.uint32))
    assert 0 < refused < 32


@pytest.mark.parametrize("span", [200, 2**31 - 10])
@pytest.mark.parametrize("value", ["i32", "f32"])
@pytest.mark.parametrize("labels", ["i32", "i64", "u32"])
def test_readout_of_hash_tables(span, value, labels):
    """Unsorted relations of every key width and value type, read to host and to
    device buffers aligned only to the element size."""
    import ctypes as C

    import torch

    from paper_2609_27203_amd import xlh
    print(f"case: hash table readout span={span} value={value} labels={labels}", flush=True)
    rng = np.random.default_rng(span & 0xffff)
    n = 20_000
    kt = {"i32": np.int32, "i64": np.int64, "u32": np.uint32}[labels]
    a = rng.integers(0, span, n).astype(kt)
    b = rng.integers(0, span, n).astype(kt)
    v = (rng.integers(-10**6, 10**6, n) if value == "i32" else rng.standard_normal(n)).astype(
        np.int32 if value == "i32" else np.float32)
    ctx = xlh.Context(device=0, workspace_bytes=512 << 20)
    ctx.set_option("index_mode", 1)
    ctx.set_option("hash_min_log2", 16)
    ctx.relation("e", (labels, labels, value)).load([a, b, v])
    ctx.relation("best", (labels, labels, value))
    ctx.relation("pair", (labels, labels))
    ctx.compile("best(X,Y,max(V)) :- e(X,Y,V).\npair(Y,X) :- e(X,Y,_).").run()
    order = np.lexsort((v, b, a))
    last = np.ones(n, bool)
    last[:-1] = (a[order][1:] != a[order][:-1]) | (b[order][1:] != b[order][:-1])
    want = {"best": [c[order][last] for c in (a, b, v)]}
    want["pair"] = _canonical([b, a])
    for name, cols in want.items():
        rel, m = ctx.relations[name], len(cols[0])
        assert rel.size() == m
        for g, w in zip(rel.read(), cols):
            assert np.array_equal(g, w)
        for shift in (0, 1):
            bufs = [torch.full(((m + 2) * c.itemsize,), 0x5A, dtype=torch.uint8, device="cuda") for c in cols]
            ptrs = (C.c_void_p * len(cols))(*[x.data_ptr() + (shift if j else 0) for j, x in enumerate(bufs)])
            got = C.c_int64()
            ctx._check(xlh.lib().xl_relation_read(rel._h, ptrs, m, C.byref(got), 1))
            for j, (x, w) in enumerate(zip(bufs, cols)):
                at = shift if j else 0
                assert np.array_equal(x.cpu().numpy()[at:at + w.nbytes], w.view(np.uint8))
    ctx.close()


@pytest.mark.parametrize("name", list(WIDTHS))
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1000, 3071])
def test_small_loads(name, n):
    """Loads of one workgroup: every column layout, duplicates, rows of one value."""
    types, make = WIDTHS[name]
    cols = make(np.random.default_rng(n), n)
    cols = [np.ascontiguousarray(np.r_[c, c[: len(c) // 3]])[:4096] for c in cols]
    want = _canonical_bits(cols)
    for device, shift in ((False, 0), (True, 0), (True, 2)):
        print(f"case: small load {name} n={n} device={device} shift={shift}", flush=True)
        for g, w in zip(_load_and_read(types, cols, device, shift, 8 << 20), want):
            assert np.array_equal(g.view(np.uint32), w.view(np.uint32))


@pytest.mark.parametrize("value", ["f32", "narrow", "few", "same"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("run", [1, 2, 63, 64, 65, 66, 129, 2047, 2049, 20_000])
def test_payload_order_within_runs(run, wide, value):
    """Rows that agree in all columns but the payload, in runs around the length
    that is ordered by counting and around a tile of rows: keys of 32 and 64 bits."""
    rng = np.random.default_rng(run)
    n = 20_011
    at = np.arange(n) // run
    a = (at * (2**31 // (n // run + 2)) if wide else at * (2**12 // (n // run + 2) or 1) % 2**12)
    b = rng.integers(0, 2**31 - 1 if wide else 2**12, at[-1] + 1)[at]
    a, b = np.r_[0, 2**31 - 1 if wide else 2**12 - 1, a], np.r_[0, 2**31 - 1 if wide else 2**12 - 1, b]
    v = {"f32": rng.standard_normal(n + 2), "narrow": rng.integers(-2**19, 2**19, n + 2),
         "few": rng.integers(0, 3, n + 2) * 2**20, "same": np.where(np.arange(n + 2) < 2, 2**24, 7)}[value]
    cols = [a.astype(np.int32), b.astype(np.int32), v.astype(np.float32 if value == "f32" else np.int32)]
    order = rng.permutation(n + 2)
    cols = [np.ascontiguousarray(c[order]) for c in cols]
    types = ("i32", "i32", "f32" if value == "f32" else "i32")
    want = _canonical_bits(cols)
    for device in (False, True):
        print(f"case: runs of {run} wide={wide} value={value} device={device}", flush=True)
        for g, w in zip(_load_and_read(types, cols, device), want):
            assert np.array_equal(g.view(np.uint32), w.view(np.uint32))


def test_long_runs_in_a_workspace_that_holds_less():
    """Smaller workspaces down to one that refuses the load: the rows are right or the call is refused."""
    from paper_2609_27203_amd import xlh
    types, make = WIDTHS["payload_long_run"]
    cols = make(np.random.default_rng(2), 50_000)
    want = _canonical_bits(cols)
    refused = 0
    for ws in [(1 << 20) + i * (1 << 17) for i in range(24)]:
        print(f"case: long runs loaded in {ws} bytes", flush=True)
        for device in (False, True):
            try:
                got = _load_and_read(types, cols, device, 0, ws)
            except xlh.XlError as e:
                assert e.status_name == "XL_RESOURCE_EXHAUSTED"
                refused += 1
                continue
            for g, w in zip(got, want):
                assert np.array_equal(g.view(np.uint32), w.view(np.uint32))
    assert 0 < refused < 48
