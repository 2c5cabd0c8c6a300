"""Plans under a scratch limit (cronus_attn_mixed_static's array) and lean plans (a workspace of versions up
to 505), under the sanitizers: they cover every row and key like any other plan, a batch that fits
in the limit with its tiles whole fits in it whatever cut and span are taken."""
import numpy as np

from paper_2509_17357_amd import workloads as W

import test_plan_cpu as TP
from test_plan_sanitized_cpu import exe, plan_line, run_cases  # noqa: F401 (fixture)

SHAPES = [W.HeadShape(32, 8, 128), W.HeadShape(28, 4, 128), W.HeadShape(64, 8, 128, "fp8"), W.HeadShape(8, 2, 64),
          W.HeadShape(64, 1, 128)]
LIMITS = [1 << 20, 4 << 20, 12 << 20, 64 << 20]


def batches():
    for seed in range(60):
        rng = np.random.default_rng([seed, 0x11317])
        shape = SHAPES[seed % len(SHAPES)]
        n, m = int(rng.integers(1, 4)), int(rng.integers(0, 24))
        P = np.concatenate([rng.integers(0, 9000, n), rng.integers(200, 8000, m)])
        C = np.concatenate([rng.integers(100, 700, n), np.ones(m, dtype=np.int64)])
        yield shape, P, C


def size(rep):
    return rep["image_bytes"] + rep["total_bytes"]


def test_limited_and_lean_plans(exe):  # noqa: F811
    lines, meta = [], list(batches())
    for shape, P, C in meta:
        line = plan_line(shape, 256, 0, P.tolist(), C.tolist())
        lines += [line, line.replace("plan", "lean", 1), line.replace("plan", "limited 1", 1)]
        lines += [line.replace("plan", f"limited {x}", 1) for x in LIMITS]
    replies = run_cases(exe, lines)
    per, cut_finer, tight = 3 + len(LIMITS), 0, 0
    assert len(replies) == per * len(meta)
    for i, (shape, P, C) in enumerate(meta):
        best, lean, least, *limited = replies[per * i:per * (i + 1)]
        for rep in (lean, least, *limited):
            assert rep["rc"] == 0
        for rep in (lean, least, limited[i % len(limited)]):
            TP.verify_items(shape, P, C, rep["items"], rep["stats"])
        assert size(least) <= size(lean)   # whole tiles, narrow spans by the one rule
        for x, rep in zip(LIMITS, limited):
            if size(least) <= x:
                assert size(rep) <= x, (i, x)
                cut_finer += size(least) < size(rep) < size(best)
                tight += size(best) > x
    assert cut_finer > 5 and tight > 20
