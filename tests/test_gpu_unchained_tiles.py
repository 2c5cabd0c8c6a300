"""Chunk tiles with no successor reserved: a launch with fewer items per queue than two for every
CU never asks ahead, so each of its tiles leaves with an empty mailbox, which every wave of the
work-group has to have read before the next record is written to it.  Tiles of one to a few K/V
tiles, so that the exits dominate; decodes in the same queues; both cache types and head sizes.
Every case runs many times and must give the same bits."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, kv_dtype, chunk sequences, chunk range, prefix range, decodes)
    (32, 8, 128, "bf16", 36, (33, 128), (0, 40), 6),    # tiles of one to three K/V tiles
    (28, 4, 128, "bf16", 60, (40, 90), (0, 250), 9),    # ragged tails
    (8, 2, 64, "bf16", 150, (33, 64), (0, 60), 5),
    (64, 8, 128, "fp8", 40, (17, 60), (0, 200), 6),     # codes converted on the way
    (8, 2, 64, "fp8", 150, (33, 64), (0, 60), 5),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tiles_without_a_reserved_successor(case):
    hq, hkv, d, dt, n, chunk, prefix, decodes = CASES[case]
    rng = np.random.default_rng(8100 + case)
    C = rng.integers(chunk[0], chunk[1], size=n, endpoint=True).tolist() + [1] * decodes
    P = rng.integers(prefix[0], prefix[1], size=n, endpoint=True).tolist() + rng.integers(1, 400, size=decodes).tolist()
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=8100 + case)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    items = B.cronus_attn_mixed_plan_items(it.cache, batch.prefix_lens, batch.chunk_lens)
    per_queue = np.bincount(items[:, 10], minlength=8)
    assert 32 < per_queue.max() < 96 and (items[:, 9] >= 1).sum() > 256  # more than one tile a CU, never two more per CU left
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    for k in range(64):
        it.out.zero_()
        it.attention()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out), k
