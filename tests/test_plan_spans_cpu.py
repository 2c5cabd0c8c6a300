"""Key spans of decodes: one length for the whole launch, the narrow items' keys over the CUs in
whole steps of 256, from 512 to 4096; a row's keys in equal spans of at most that length and a
quarter of it, in whole steps.  The cut decides the bits of a result (the running reference and
the order of the sums): a decode-only iteration takes this one rule and no other."""
import numpy as np
import pytest

from paper_2509_17357_amd import workloads as W

from test_plan_cpu import F, plan_for

CUS = 256  # what the planner assumes without a device


def up(x, step):
    return -(-x // step) * step


@pytest.mark.parametrize("n, lo, hi", [(16, 200, 3000), (5, 50, 900), (20, 1500, 2500), (31, 100, 700), (33, 300, 4000), (128, 500, 500),
                                       (3, 9000, 30000)])
def test_decode_spans_follow_the_rule(n, lo, hi):
    rng = np.random.default_rng([n, lo, hi])
    for sh in (W.SHAPE_8B, W.HeadShape(28, 4, 128), W.HeadShape(8, 2, 64)):
        L = rng.integers(lo, hi, size=n, endpoint=True)
        items, _ = plan_for(sh, L - 1, np.ones(n, dtype=int))
        span = min(max(up(-(-int(L.sum()) * sh.n_kv_heads // CUS), 256), 512), 4096)
        for s in range(n):
            k = max(1, -(-int(L[s]) // span))
            if k > 1 and L[s] - (k - 1) * span <= span // 4:
                k -= 1
            per = up(-(-int(L[s]) // k), 256)
            of_row = items[(items[:, F["seq"]] == s) & (items[:, F["kv_head"]] == 0)]
            begins = np.sort(of_row[:, F["kv_begin"]])
            assert begins.tolist() == list(range(0, int(L[s]), per))
            assert of_row[:, F["kv_end"]].max() == L[s]
