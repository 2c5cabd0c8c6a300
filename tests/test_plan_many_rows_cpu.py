"""More rows to cut than a launch has arrival counters (4096): the longest rows are cut, so that
no row of a length that matters is left whole behind the others.  The list is run through the
order in which work-groups take items (own queue, then the others) with the planner's own
estimate of a narrow item's time, 9.6 us + 14.1 ns a key; the end must be near the mean."""
import heapq

import numpy as np
import pytest

from paper_2509_17357_amd import workloads as W

from test_plan_cpu import F, plan_for, verify_items


def scheduled_end(items, cus=256):
    """(end, sum of the items' times / CUs), in us, for 8 queues of cus / 8 work-groups each."""
    t = 9.6 + 0.0141 * (items[:, F["kv_end"]] - items[:, F["kv_begin"]])
    queues = [t[items[:, F["queue"]] == x].tolist() for x in range(8)]
    head = [0] * 8
    free = [(0.0, g) for g in range(cus)]
    end = 0.0
    while free:
        now, g = heapq.heappop(free)
        for k in range(8):
            x = (g + k) % 8
            if head[x] < len(queues[x]):
                done = now + queues[x][head[x]]
                head[x] += 1
                end = max(end, done)
                heapq.heappush(free, (done, g))
                break
    return end, t.sum() / cus


CASES = {
    "one long at the end": (W.SHAPE_8B, [8000] * 512 + [128000]),
    "one long in front": (W.SHAPE_8B, [128000] + [8000] * 512),
    "four long": (W.SHAPE_8B, [8000] * 516 + [60000] * 4),
    "a million keys": (W.SHAPE_8B, [6000] * 520 + [1000000]),
    "all long": (W.SHAPE_8B, [131000] * 600),
    "twice as many as counters, ragged": (W.SHAPE_8B, np.random.default_rng(5).integers(5000, 70000, 1100).tolist()),
    "four KV heads": (W.HeadShape(28, 4, 128), [7000] * 1030 + [300000] * 2),
    "three KV heads": (W.HeadShape(12, 3, 64), [7000] * 1500 + [250000] * 3),
    "two head groups": (W.HeadShape(48, 1, 64), [9000] * 2100 + [400000]),
}


@pytest.mark.parametrize("name", CASES)
def test_long_rows_are_cut_first(name):
    shape, L = CASES[name]
    P, C = np.array(L) - 1, np.ones(len(L), dtype=int)
    items, stats = plan_for(shape, P, C)
    verify_items(shape, P, C, items, stats)
    per_row = shape.n_kv_heads * -(-shape.n_q_heads // shape.n_kv_heads // 32)
    assert 4096 - per_row < stats["merge_groups"] <= 4096
    keys = items[:, F["kv_end"]] - items[:, F["kv_begin"]]
    whole = items[:, F["partial"]] < 0
    cut_rows = np.unique(items[~whole][:, F["seq"]])
    left = np.array(L)[np.setdiff1d(np.arange(len(L)), cut_rows)]
    assert left.max() <= np.array(L)[cut_rows].min()
    # left whole: an item no longer than 4096 - per_row others' keys, at most 1/15 of a CU's share
    assert keys.max() <= keys.sum() / 256 / 15
    for x in range(8):  # and such items are taken first, longest first
        q = keys[items[:, F["queue"]] == x]
        over = q > 5120
        assert not over[over.sum():].any() and (np.diff(q[:over.sum()]) <= 0).all()
    end, mean = scheduled_end(items)
    assert end <= 1.03 * mean, (end, mean)


def test_rows_next_to_chunks():
    """Tiles that are cut into spans keep their counters; the decodes share the rest."""
    rng = np.random.default_rng(11)
    L = rng.integers(5200, 9000, 560)
    P, C = np.concatenate([[60000], L - 1, [90000]]), np.concatenate([[480], np.ones(560, dtype=int), [1]])
    items, stats = plan_for(W.SHAPE_8B, P, C)
    assert 4096 - 8 - 64 < stats["merge_groups"]
    wide = items[:, F["wide"]] >= 1
    cut = len(np.unique(items[wide & (items[:, F["partial"]] >= 0)][:, [F["kv_head"], F["q_tok0"]]], axis=0))
    narrow_cut = items[~wide & (items[:, F["partial"]] >= 0)]
    assert cut + len(np.unique(narrow_cut[:, [F["seq"], F["kv_head"]]], axis=0)) <= 4096
    assert 561 in narrow_cut[:, F["seq"]]
