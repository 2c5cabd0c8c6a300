"""Wide tiles that a work-group runs back to back while its queue is well filled: the next
tile's record, table entries, first K/V tiles and Q are requested before the finished tile is
stored.  Checked where that can go wrong: tiles of one K/V tile and of many (the record arrives
before, at or behind the last hand-over), tiles whose rows end inside a wave's share, one head
per group, D = 64, the bf16 copy of an fp8 cache, chunks behind a prefix, decodes in the same
queues; every case runs several times and must give the same bits."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, kv_dtype, sequences, chunk range, prefix range, decodes)
    (32, 8, 128, "bf16", 48, (40, 640), (0, 0), 0),    # whole prompts of 1 .. 10 K/V tiles
    (28, 4, 128, "bf16", 48, (40, 700), (0, 90), 9),   # 252-row tiles, ragged tails, decodes
    (8, 8, 128, "bf16", 40, (200, 900), (0, 0), 3),    # one head per group: 256 tokens per tile
    (8, 2, 64, "bf16", 150, (33, 500), (0, 40), 5),    # D = 64
    (16, 2, 128, "fp8", 40, (512, 560), (0, 30), 6),   # tiles that read the bf16 copy
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tiles_run_back_to_back(case):
    hq, hkv, d, dt, n, chunk, prefix, decodes = CASES[case]
    rng = np.random.default_rng(7300 + case)
    C = rng.integers(chunk[0], chunk[1], size=n, endpoint=True).tolist() + [1] * decodes
    P = rng.integers(prefix[0], prefix[1], size=n, endpoint=True).tolist() + rng.integers(1, 900, size=decodes).tolist()
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=7300 + case)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    items = B.cronus_attn_mixed_plan_items(it.cache, batch.prefix_lens, batch.chunk_lens)
    assert np.bincount(items[:, 10], minlength=8).max() >= 96  # three items per CU of an XCD: tiles are chained
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    for _ in range(4):
        it.out.zero_()
        it.attention()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out)
