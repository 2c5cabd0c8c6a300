"""The work list in the kernel's arguments: decode batches whose compact list (48 bytes a sequence of 8 KV heads) is just
below and above the two sizes that the arguments come in, 1280 and 3840 bytes; tiles, tile spans and a row of many spans in
such lists.  Each with a workspace and without one (the same bits), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

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
