"""The work list in the kernel's arguments: decode batches whose compact list (48 bytes a sequence of 8 KV heads) is just
below and above the two sizes that the arguments come in, 1280 and 3840 bytes; tiles, tile spans and a row of many spans in
such lists.  Each with a workspace and without one (the same bits), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu
G7, MHA = W.HeadShape(28, 4, 128), W.HeadShape(8, 8, 64)


@pytest.mark.parametrize("shape, P, C", [(MHA, [90 + 7 * i for i in range(26)], [1] * 26), (MHA, [90 + 7 * i for i in range(27)], [1] * 27),
                                         (MHA, [20 + i for i in range(80)], [1] * 80), (MHA, [20 + i for i in range(81)], [1] * 81),
                                         (W.HeadShape(16, 2, 64, "fp8"), [700, 40, 0], [70, 1, 33]),
                                         (G7, [3000, 6000, 5], [90, 1, 40]), (W.HeadShape(8, 4, 64), [60000] + [10] * 64, [1] * 65)])
def test_lists_in_and_beyond_the_arguments(shape, P, C):
    batch = W.custom_batch(shape, P, C, seed=9950 + len(P))
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    for _ in range(2):
        it.out.zero_()
        B.cronus_attn_mixed_static(it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks,
                                   it.sm_scale, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out)


WIDE = {"bf16, D 64": (W.HeadShape(32, 32, 64), [0] * 39, [200] * 39),
        "fp8, D 64": (W.HeadShape(32, 32, 64, "fp8"), [0, 40, 7] * 13, [190, 70, 130] * 13),
        "bf16, D 128, prompts of one to four key tiles, then decodes": (W.HeadShape(32, 32, 128), [0] * 30 + [300, 5, 64, 700, 33, 128], [200, 70, 130, 256, 33, 64] * 5 + [1] * 6),
        "fp8, D 128, decodes between": (W.HeadShape(32, 32, 128, "fp8"), [0, 0, 90, 10, 0, 400] * 6, [140, 33, 100, 250, 60, 1] * 6)}


@pytest.mark.parametrize("name", WIDE)
def test_tiles_taken_ahead_from_a_list_in_the_arguments(name):
    """Many wide items in a list that the arguments hold: a work-group asks for its next item while it works on a tile, as long as
    its queue holds another item for each of the 32 work-groups of its XCD after the first round, and goes over to it without a pause."""
    shape, P, C = WIDE[name]
    batch = W.custom_batch(shape, P, C, seed=9800 + len(name))
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    items = B.cronus_attn_mixed_plan_items(it.cache, batch.prefix_lens, batch.chunk_lens)
    col = {f: items[:, i] for i, f in enumerate(B.PLAN_ITEM_FIELDS)}
    units = len({tuple(x) for x in items[col["kv_head"] == 0][:, [0, 4]].tolist()})
    assert 1280 < 32 * units + 2 * len(items) <= 3840  # a list of the larger size
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    for x in range(8):
        wide = (col["queue"] == x) & (col["wide"] > 0)
        # after the static items, and the 2 x 32 that have to be left, tiles are still to come
        assert (col["queue"] == x).sum() - n_cus // 8 - 2 * (n_cus // 8) >= 8 and wide.sum() > n_cus // 8
    for _ in range(2):
        it.out.zero_()
        B.cronus_attn_mixed_static(it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks,
                                   it.sm_scale, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out)


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape, n, P, C", [((32, 32, 64), 8, 8000, 256), ((32, 8, 128), 7, 9000, 256)])
def test_long_tiles_from_a_list_in_the_arguments(kv_dtype, shape, n, P, C):
    """Uncut tiles of more than 250 key sub-tiles in a list of either size: the steady loops of the kernels that take one give the
    bits of those that read records, which other tests hold against the oracle."""
    it = DeviceIteration(W.custom_batch(W.HeadShape(*shape, kv_dtype), [P] * n, [C] * n, seed=9900), pool_fill=0)
    it.load_device_inputs()
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.step()
    torch.cuda.synchronize()
    want = bits_from_bf16_tensor(it.out).copy()
    b = it.batch
    items = B.cronus_attn_mixed_plan_items(it.cache, b.prefix_lens, b.chunk_lens)
    units = len({tuple(x) for x in items[items[:, 1] == 0][:, [0, 4]].tolist()})
    assert (items[:, 9] == 1).all() and (items[:, 7] - items[:, 6] > 32 * 250).all()
    assert (32 * units + 2 * len(items) <= 1280) == (shape[2] == 64) and 32 * units + 2 * len(items) <= 3840
    for _ in range(4):
        it.out.zero_()
        B.cronus_attn_mixed_static(it.cache, it.q, it.out, b.prefix_lens, b.chunk_lens, it.block_tables, b.max_blocks, it.sm_scale,
                                   torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), want)
