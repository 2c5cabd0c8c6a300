"""Results of key spans are merged by the main kernel itself: the wave that arrives last
combines its rows' spans.  Checked where the merge can go wrong: two spans and many (more than
one group of four loads), one row and 32, rows that end inside a wave's share, both head
sizes and cache types, tiles cut into spans; every case runs several times, since a launch must
leave every arrival counter at zero for the next, and must give the same bits each time
(spans are combined in order, whoever arrives last)."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, kv_dtype, prefix_lens, chunk_lens)
    (1, 1, 128, "bf16", [4096, 0], [1, 3]),                # two spans of one row
    (8, 1, 64, "bf16", [33000], [1]),                      # nine spans of 8 rows, D = 64
    (32, 1, 128, "bf16", [5000, 1029], [1, 1]),            # 32 rows: two passes over the rows
    (28, 4, 128, "bf16", [4500, 600], [4, 1]),             # 28 rows of four tokens: the last wave's share is short
    (16, 2, 128, "fp8", [9000, 1023], [1, 2]),             # fp8 decodes and a short chunk, merged
    (8, 2, 64, "fp8", [3000], [100]),                      # a tile cut into spans, converted on the fly, D = 64
    (32, 8, 128, "bf16", [9000, 2000], [65, 1]),           # tile spans, and a narrow tail of one token
    (8, 2, 64, "bf16", [7000], [90]),                      # tile spans, D = 64, a tile with rows for three waves
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_merged_spans_match_the_oracle_every_time(case):
    hq, hkv, d, dt, P, C = CASES[case]
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=9400 + case)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    assert B.cronus_attn_mixed_plan_stats(it.cache, batch.prefix_lens, batch.chunk_lens)["merge_groups"] > 0
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    for _ in range(12):  # more calls than there are sets of counters
        it.out.zero_()
        it.attention()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out)
