"""fp8 chunk tiles that convert codes on their way into LDS, run back to back: the next tile's codes
are requested three tiles ahead and its Q before the finished rows are stored.  Tiles of one to
many K/V tiles (fewer than the ring holds, as many, more), rows that end inside a wave's share,
both head sizes, several head groupings; and queues in which such tiles alternate with tiles
that read the bf16 copy, where one kind may not reserve the other.  Every case runs several
times and must give the same bits."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, [(sequences, chunk range, prefix range)], decodes, kinds of tiles: 1 codes, 2 copy)
    (16, 2, 128, [(60, (40, 480), (0, 400))], 6, {1}),                        # 1 .. 14 K/V tiles
    (16, 2, 128, [(120, (33, 250), (0, 0)), (3, (470, 470), (1500, 1700))], 0, {1}),  # short ones, a few long
    (28, 4, 128, [(60, (60, 250), (0, 200))], 9, {1}),                        # 252-row tiles
    (8, 2, 64, [(90, (65, 600), (0, 300))], 5, {1}),
    (8, 8, 64, [(70, (257, 700), (0, 100))], 3, {1}),                         # one head per group
    (16, 2, 128, [(40, (60, 480), (0, 300)), (12, (520, 620), (0, 200))], 6, {1, 2}),
    (8, 2, 64, [(60, (65, 600), (0, 300)), (6, (1030, 1200), (0, 100))], 6, {1, 2}),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_code_tiles_run_back_to_back(case):
    hq, hkv, d, chunks, decodes, kinds = CASES[case]
    rng = np.random.default_rng(8500 + case)
    C = np.concatenate([rng.integers(c[0], c[1], size=n, endpoint=True) for n, c, p in chunks])
    P = np.concatenate([rng.integers(p[0], p[1], size=n, endpoint=True) for n, c, p in chunks])
    order = rng.permutation(C.size)
    C, P = C[order].tolist() + [1] * decodes, P[order].tolist() + rng.integers(1, 900, size=decodes).tolist()
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, "fp8"), P, C, seed=8500 + case)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    items = B.cronus_attn_mixed_plan_items(it.cache, batch.prefix_lens, batch.chunk_lens)
    wide = items[items[:, 9] >= 1]
    assert set(np.minimum(wide[:, 9], 2).tolist()) == kinds
    # three items per CU of an XCD and more: tiles are reserved ahead
    assert np.bincount(wide[:, 10], minlength=8).min() >= 96
    if kinds == {1, 2}:
        for x in range(8):
            kind = np.minimum(wide[wide[:, 10] == x][:, 9], 2)
            assert (np.diff(kind) != 0).any()
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
    for k in range(6):
        it.out.zero_()
        it.attention()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), out), k
