"""logsumexp over infinite values: a fold with +inf among its terms is +inf, one
of -inf alone is -inf."""
import numpy as np
import pytest

from helpers import LSE_TOL, engine_run
from paper_2609_27203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batched_rounds", [0, 4])
@pytest.mark.parametrize("sources", [1, 40, 64, 130])
def test_one_infinite_term_in_a_pull(sources, batched_rounds):
    """A target's terms from up to 20 middle nodes, one of them +inf: dense pulls
    of short lists.  Finite keys are folded by numpy in 64 bits."""
    lists = [[np.inf], [0, np.inf, 1], [np.inf, -3], [-3, np.inf], [-np.inf, np.inf], [-1] * 9 + [np.inf] + [2] * 8,
             [np.inf] + [0] * 19, [-np.inf], [-np.inf, 1], [-np.inf] * 9, [1, 2, 3]]
    mids = 20
    src, dst, w = [], [], []
    for s in range(sources):
        src += [s] * mids
        dst += list(range(200, 200 + mids))
        w += [0.0] * mids
    for t, terms in enumerate(lists):
        src += list(range(200, 200 + len(terms)))
        dst += [300 + t] * len(terms)
        w += terms
    src, dst, w = np.int32(src), np.int32(dst), np.float32(w)
    wl = W.Workload("lse", W.LSE_RULES, {"edge": (("i32", "i32", "f32"), [src, dst, w]),
                                         "source": (("i32",), [np.arange(sources, dtype=np.int32)])},
                    {"score": ("i32", "i32", "f32")})
    print(f"case: one infinite term sources={sources} batched_rounds={batched_rounds}", flush=True)
    rels, stats, _ = engine_run(wl, options={"batched_rounds": batched_rounds, "profile": 1})
    assert stats["pull_launches"] > 0
    s, y, p = rels["score"]
    assert len(s) == sources * (mids + len(lists))
    for t, terms in enumerate(lists):
        got, x = p[y == 300 + t], np.float64(terms)
        m = x.max()
        want = m if np.isinf(m) else m + np.log(np.exp(x - m).sum())
        assert len(got) == sources
        assert np.all(got == want) if np.isinf(m) else np.all(np.abs(got - want) <= LSE_TOL * max(1, abs(want)))
