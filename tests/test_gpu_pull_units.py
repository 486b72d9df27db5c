"""Pulls straight from the mark words: units of eight and of two words, short and long in-edge lists."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

I2F = ("i32", "i32", "f32")
RULES = """
h(S,Y,logsumexp(W)) :- u(S), d(S,Y,W).
h(S,Y,logsumexp(D)) :- h(S,Z,P), d(Z,Y,W), D is P + W.
"""


# width 2,000: about 50,000 mark words, more than the 32,768 of a small head; long:
# the share of targets with 40 in-edges (the others have 1 to 8)
@pytest.mark.parametrize("width,sources", [(40, 3), (300, 64), (2000, 225), (2000, 256)])
@pytest.mark.parametrize("long", [0.0, 0.02, 0.5, 1.0])
def test_layers(width, sources, long):
    from paper_2609_27203_amd import xlh
    print(f"case: pull units width={width} sources={sources} long={long}", flush=True)
    rng = np.random.default_rng(width + sources)
    layers = 3
    sources = min(sources, width)
    src, dst, wgt = [], [], []
    # base edges from the sources (their own scores stay absent), then layer to layer
    score = np.full((sources, width), -np.inf)
    for s in range(sources):
        for y in rng.integers(0, width, 6):
            src.append(s), dst.append(sources + y), wgt.append(rng.uniform(-3, 0))
    src, dst, wgt = [np.array(x) for x in (src, dst, np.float32(wgt))]
    pair = np.unique(src * 10**6 + dst, return_index=True)[1]
    src, dst, wgt = src[pair], dst[pair], wgt[pair]
    score[src, dst - sources] = wgt.astype(np.float64)
    edges, want = [(src, dst, wgt)], {}
    for layer in range(layers):
        first = sources + layer * width
        for s, y in zip(*np.nonzero(np.isfinite(score))):
            want[(int(s), first + int(y))] = score[s, y]
        if layer == layers - 1:
            break
        deg = np.where(rng.random(width) < long, 40, rng.integers(1, 9, width))
        y = np.repeat(np.arange(width), deg)
        key = np.unique(y * width + rng.integers(0, width, len(y)))
        y, z = key // width, key % width
        w = rng.uniform(-3, 0, len(y)).astype(np.float32)
        edges.append((first + z, first + width + y, w))
        at = np.searchsorted(y, np.arange(width))
        score = np.logaddexp.reduceat(score[:, z] + w.astype(np.float64), at, axis=1)
    cols = [np.concatenate([e[j] for e in edges]) for j in range(3)]
    ctx = xlh.Context(device=0, workspace_bytes=4 << 30)
    ctx.relation("d", I2F).load([cols[0].astype(np.int32), cols[1].astype(np.int32), cols[2]])
    ctx.relation("u", ("i32",)).load([np.arange(sources, dtype=np.int32)])
    ctx.relation("h", I2F)
    ctx.compile(RULES).run()
    s, y, v = ctx.relations["h"].read()
    ctx.close()
    keys = sorted(want)
    assert [(int(a), int(b)) for a, b in zip(s, y)] == keys
    ref = np.array([want[k] for k in keys])
    assert np.all(np.abs(v - ref) <= 1e-5 * np.maximum(1, np.abs(ref)))
