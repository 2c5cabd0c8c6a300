"""Decodes read K/V non-temporally unless a neighbour in the batch has the same block: the same keys give the same bits from
blocks of their own, from shared ones (all of them, the last span's, every fourth sequence's) and for head groups that share a KV head."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, n, keys", [(W.SHAPE_8B, 20, 701), (W.SHAPE_8B, 3, 5000), (W.HeadShape(16, 2, 128, "fp8"), 18, 1300),
                                            (W.HeadShape(8, 4, 64), 33, 33), (W.HeadShape(64, 1, 128), 5, 900)])
def test_shared_blocks_give_the_same_bits(shape, n, keys):
    it = DeviceIteration(W.custom_batch(shape, [keys - 1] * n, [1] * n, seed=9700 + n), pool_fill=0x5A)
    it.load_device_inputs()
    for t in (it.ctx_k, it.ctx_v, it.new_k, it.new_v):
        rows = t.view(n, -1)
        rows[1:] = rows[:1]
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.setup_decode_context()
    it.step()
    torch.cuda.synchronize()
    want = bits_from_bf16_tensor(it.out).copy()
    assert np.any(want)
    own = it.block_tables.clone()
    blocks = (keys + 15) // 16
    for rows, cols in ((slice(None), slice(0, blocks)), (slice(None), slice(blocks // 2, blocks)), (slice(None, None, 4), slice(0, blocks))):
        it.block_tables.copy_(own)
        it.block_tables[rows, cols] = own[0, cols]
        it.out.zero_()
        it.attention()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), want)
