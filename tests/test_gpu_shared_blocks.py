"""Decodes read K/V non-temporally unless a neighbour in the batch has the same block: the same keys give the same bits from
blocks of their own, from shared ones (all of them, the last span's, every fourth sequence's) and for head groups that share a KV head."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
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


@pytest.mark.parametrize("shape, n, keys", [(W.SHAPE_8B, 33, 701), (W.HeadShape(16, 8, 128, "fp8"), 36, 1300), (W.HeadShape(8, 4, 64), 90, 1000)])
def test_shared_blocks_of_large_launches(shape, n, keys):
    """The same where the launch's K/V is large enough (90 MB) to be read non-temporally at all, with the records in host memory
    and with the list in the arguments."""
    assert n * keys * 2 * shape.n_kv_heads * shape.head_dim * (1 if shape.kv_dtype == "fp8" else 2) >= 90e6
    it = DeviceIteration(W.custom_batch(shape, [keys - 1] * n, [1] * n, seed=9750 + n), pool_fill=0x5A)
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
    own, b = it.block_tables.clone(), it.batch
    blocks = (keys + 15) // 16
    for rows, cols in ((slice(0, 0), slice(0, 0)), (slice(None), slice(0, blocks)), (slice(None), slice(blocks // 2, blocks)),
                       (slice(None, None, 9), slice(0, blocks)), (slice(None, None, 8), slice(0, blocks))):
        it.block_tables.copy_(own)
        it.block_tables[rows, cols] = own[0, cols]
        for static in (False, True):
            it.out.zero_()
            if static:
                B.cronus_attn_mixed_static(it.cache, it.q, it.out, b.prefix_lens, b.chunk_lens, it.block_tables, b.max_blocks, it.sm_scale,
                                           torch.cuda.current_stream().cuda_stream)
            else:
                it.attention()
            torch.cuda.synchronize()
            assert np.array_equal(bits_from_bf16_tensor(it.out), want), (rows, cols, static)
