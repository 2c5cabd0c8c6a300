"""Batches at the limit of cronus_attn_mixed_static's array.  The limit is checked on the host
before the device is looked at, so without a GPU a batch that fits ends with the HIP error of
the set-up and one that does not with WORKSPACE; both before anything is launched."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B, workloads as W

from test_plan_cpu import plan_for

SLOT_BYTES = 32 * (128 + 2) * 4  # fp32 O, m and l of 32 rows


def call(shape, P, C):
    cache = B.make_cache(1 << 20, 1 << 24, 1 << 20, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, B.CRONUS_KV_BF16)
    P, C = np.asarray(P, dtype=np.int32), np.asarray(C, dtype=np.int32)
    try:
        B.cronus_attn_mixed_static(cache, 1 << 28, 1 << 29, P, C, 1 << 30, int((P + C).max() + 15) // 16, 0.1, 0)
    except B.CronusError as e:
        return e.status
    return B.CRONUS_OK


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")
@pytest.mark.parametrize("decodes, over, fits", [([], True, True), ([5000] * 8, True, True), ([5000] * 16, True, True),
                                                 ([5000] * 50, False, True), ([40000] * 128, True, False)])
def test_tiles_are_cut_coarser_before_a_batch_is_refused(decodes, over, fits):
    shape = W.HeadShape(64, 8, 128)
    # (tiles of nearly one length, which the planner cuts)
    P, C = [6948, 3291, 3262] + decodes, [1128, 564, 125] + [1] * len(decodes)
    _, stats = plan_for(shape, P, C)
    assert (stats["partials"] * SLOT_BYTES > 64 << 20) == over  # the fastest cut
    assert (call(shape, P, C) != B.CRONUS_ERR_WORKSPACE) == fits
