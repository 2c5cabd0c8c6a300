"""A launch has arrival counters for 4096 merge groups: the planner splits no further rows
once they are used up, and still covers every key."""
import numpy as np
import pytest

from paper_2509_17357_amd import workloads as W

from test_plan_cpu import F, plan_for


@pytest.mark.parametrize("n_seqs", [512, 513, 700])
def test_split_groups_never_exceed_the_counters(n_seqs):
    sh = W.SHAPE_8B
    P, C = [7000] * n_seqs, [1] * n_seqs                     # two spans per (sequence, KV head)
    items, stats = plan_for(sh, P, C)
    assert stats["merge_groups"] == min(8 * n_seqs, 4096)
    key = items[:, F["seq"]] * 8 + items[:, F["kv_head"]]
    keys = np.bincount(key, weights=items[:, F["kv_end"]] - items[:, F["kv_begin"]], minlength=8 * n_seqs)
    assert (keys == 7001).all()
    whole = items[items[:, F["partial"]] < 0]
    assert len(whole) == 8 * n_seqs - stats["merge_groups"]
    assert (whole[:, F["kv_begin"]] == 0).all() and (whole[:, F["kv_end"]] == 7001).all()
