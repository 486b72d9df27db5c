"""Readout of relations whose rows are stored in canonical order (no sort: one
pass over the columns), through the C ABI with device destinations of every
element size, at vector-width remainders and with destinations aligned only to
the element size.  Everything is compared bit for bit."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NP = {"i32": np.int32, "f32": np.float32, "u32": np.uint32, "i64": np.int64, "u64": np.uint64, "f64": np.float64,
      "bool": np.bool_}
TYPES = [("i32", "i64", "bool", "f32"), ("u32", "f64", "u64", "i32"), ("f64",), ("bool", "bool")]


def _column(rng, t, n):
    if t == "bool":
        return rng.integers(0, 2, n).astype(bool)
    if t in ("f32", "f64"):
        return rng.standard_normal(n).astype(NP[t])
    info = np.iinfo(NP[t])
    return rng.integers(info.min, info.max, n, dtype=NP[t], endpoint=True)


def _canonical(cols):
    """Distinct rows in ascending lexicographic order (no zeros among the floats)."""
    order = np.lexsort(cols[::-1])
    cols = [c[order] for c in cols]
    keep = np.ones(len(order), bool)
    if len(order) > 1:
        keep[1:] = np.any([c[1:] != c[:-1] for c in cols], axis=0)
    return [c[keep] for c in cols]


@pytest.mark.parametrize("types", TYPES)
@pytest.mark.parametrize("n", [1, 2, 3, 5, 64, 257, 70001])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_sorted_readout(types, n, shift):
    import torch

    from paper_2609_27203_amd import xlh
    print(f"case: sorted readout {types} n={n} shift={shift}", flush=True)
    rng = np.random.default_rng(n)
    cols = [_column(rng, t, n) for t in types]
    want = _canonical(cols)
    m = len(want[0])
    ctx = xlh.Context(device=0, workspace_bytes=64 << 20)
    rel = ctx.relation("r", types)
    rel.load(cols)
    assert rel.size() == m
    sizes = [np.dtype(NP[t]).itemsize for t in types]
    # destinations that start `shift` elements into a buffer, with guards on both sides
    bufs = [torch.full(((m + shift + 2) * s,), 0x5A, dtype=torch.uint8, device="cuda") for s in sizes]
    ptrs = (C.c_void_p * len(types))(*[b.data_ptr() + shift * s for b, s in zip(bufs, sizes)])
    got = C.c_int64()
    ctx._check(xlh.lib().xl_relation_read(rel._h, ptrs, m, C.byref(got), 1))
    assert got.value == m
    for b, s, w in zip(bufs, sizes, want):
        raw = b.cpu().numpy()
        assert np.array_equal(raw[shift * s:(shift + m) * s], w.view(np.uint8))
        assert (raw[:shift * s] == 0x5A).all() and (raw[(shift + m) * s:] == 0x5A).all()
    for h, w in zip(rel.read(), want):  # host destinations
        assert np.array_equal(h.view(np.uint8), w.view(np.uint8))
    ctx.close()
