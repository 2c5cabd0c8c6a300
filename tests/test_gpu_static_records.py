"""The static entry point when the work list has no compact form (more than 255 head groups per KV
head): the records themselves are uploaded.  The results are the bits of the entry point with a
workspace, and match the oracle; again after a call whose list is compact."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [W.HeadShape(8224, 1, 64), W.HeadShape(16, 2, 64)])
def test_list_without_a_compact_form(shape):
    batch = W.custom_batch(shape, [100, 37, 1300], [1, 2, 1], seed=9900)
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
