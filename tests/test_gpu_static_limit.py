"""cronus_attn_mixed_static with a batch whose fastest cut does not fit in its array: the coarser plan
matches the oracle, and so does the next call with a batch that fits."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_coarser_plan_matches_the_oracle(dtype):
    batches = [W.custom_batch(W.HeadShape(64, 8, 128, dtype), [6948, 3291, 3262] + [5000] * 8, [1128, 564, 125] + [1] * 8, seed=31),
               W.custom_batch(W.HeadShape(64, 8, 128, dtype), [2049, 700], [201, 1], seed=32)]
    for batch, over in zip(batches, (True, False)):
        kv = U.draw_all_kv(batch)
        q = batch.gen_q()
        _, ks, vs, it = U.run_hot_path(batch, q, kv)
        stats = B.cronus_attn_mixed_plan_stats(it.cache, batch.prefix_lens, batch.chunk_lens)
        assert (stats["partials"] * 32 * (128 + 2) * 4 > 64 << 20) == over
        it.out.zero_()
        B.cronus_attn_mixed_static(it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks,
                                   it.sm_scale, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        rows = lambda s, C: np.unique(np.r_[0, C - 1, np.arange(C)[::41]])
        U.check_rows_by_sequence(batch, bits_from_bf16_tensor(it.out), q, lambda s: kv[s], it.sm_scale, ks, vs, rows_of=rows)
