"""Launches of few items carry their records in the kernel's arguments, one for each work-group, on either side of the most that fit
(48): the bits of cronus_attn_mixed_static, which goes by a list, for decodes and for chunk tiles, whole and in spans, half
tiles, queues of unequal length, both cache types and head sizes, and for iterations that place their rows in the launch."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu

ONE, ONE8, TWO, G7 = W.HeadShape(4, 1, 128), W.HeadShape(4, 1, 64, "fp8"), W.HeadShape(8, 2, 64), W.HeadShape(28, 4, 128)

CASES = {
    "one item": (ONE, [40], [1], 1),
    "47": (ONE, list(range(10, 57)), [1] * 47, 47),
    "48": (ONE, list(range(10, 58)), [1] * 48, 48),
    "49": (ONE, list(range(10, 59)), [1] * 49, 49),
    "47, fp8, D 64": (ONE8, list(range(200, 247)), [1] * 47, 47),
    "48, fp8, D 64": (ONE8, list(range(200, 248)), [1] * 48, 48),
    "49, fp8, D 64": (ONE8, list(range(200, 249)), [1] * 49, 49),
    "spans": (G7, [1300, 700], [1, 1], None),
    "a chunk and decodes": (TWO, [192, 255, 255, 255, 255], [64, 1, 1, 1, 1], 12),
    "tile spans": (TWO, [6000, 100], [60, 1], None),
    "chunks with tails": (G7, [30, 7], [50, 33], None),
    "tiles, fp8": (W.HeadShape(16, 2, 128, "fp8"), [500, 40], [90, 1], None),
    "tiles of an fp8 copy": (W.HeadShape(64, 1, 64, "fp8"), [100], [70], None),
    # the longest spans of chunk tiles in so few items (196 steps of 64 keys; of an fp8 copy, 9), in each kernel that takes records
    "long spans": (W.HeadShape(4, 1, 128), [100000], [300], 40),
    "long spans, D 64": (W.HeadShape(4, 1, 64), [100000], [300], 40),
    "long spans, fp8": (W.HeadShape(4, 1, 128, "fp8"), [100000], [300], 40),
    "long spans, fp8, D 64": (W.HeadShape(4, 1, 64, "fp8"), [100000], [300], 40),
    "long spans of an fp8 copy": (W.HeadShape(32, 1, 128, "fp8"), [1500], [128], 48),
    "long spans of an fp8 copy, D 64": (W.HeadShape(32, 1, 64, "fp8"), [1500], [128], 48),
    "skipped sequences": (TWO, [9, 100, 3], [0, 1, 0], 2),
}


@pytest.mark.parametrize("name", CASES)
def test_records_in_the_arguments(name):
    shape, P, C, n_items = CASES[name]
    it = DeviceIteration(W.custom_batch(shape, P, C, seed=13), pool_fill=0)
    it.load_device_inputs()
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.setup_decode_context()
    b = it.batch
    stats = B.cronus_attn_mixed_plan_stats(it.cache, P, C)
    assert stats["items"] == n_items if n_items else stats["items"] <= 48
    assert (stats["copy_blocks"] > 0) == ("copy" in name)
    it.place_rows()
    pools = it.k_pool.clone(), it.v_pool.clone()
    B.cronus_attn_mixed_static(it.cache, it.q, it.out, P, C, it.block_tables, b.max_blocks, it.sm_scale)
    torch.cuda.synchronize()
    want = bits_from_bf16_tensor(it.out).copy()
    for call in (it.attention, it.step, it.attention):
        it.out.zero_()
        call()
        torch.cuda.synchronize()
        got = bits_from_bf16_tensor(it.out)
        if stats["copy_blocks"] == 0:
            assert np.array_equal(got, want)
        else:  # the static entry point converts the codes itself, in another order of the sums: a bf16 step, 2^-7, at most
            f = [(x.astype(np.uint32) << 16).view(np.float32) for x in (got, want)]
            assert np.abs(f[0] - f[1]).max() <= 2.0 ** -7 * np.abs(f[1]).max()
    assert torch.equal(it.k_pool, pools[0]) and torch.equal(it.v_pool, pools[1])
