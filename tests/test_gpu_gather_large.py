"""Gathers of rows on either side of the 32 MB from which the blocks are read past the caches give back what was scattered, bit for
bit: ragged sequences that start inside a block, both head sizes, an empty one, straight after the scatter that wrote the blocks."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_kv_heads, head_dim, rows", [(8, 128, 7812), (8, 128, 7813), (8, 128, 20001), (2, 64, 62499), (2, 64, 62501)])
def test_rows_come_back(n_kv_heads, head_dim, rows):
    counts = [rows // 2 + 5, 0, 17, rows - rows // 2 - 22]
    starts = [3, 40, 0, 31]
    it = DeviceIteration(W.custom_batch(W.HeadShape(n_kv_heads, n_kv_heads, head_dim), [s + c for s, c in zip(starts, counts)], [1] * 4, seed=3),
                         pool_fill=0x11)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=it.device)
    cu, start = i32([0] + list(np.cumsum(counts))), i32(starts)
    bt, mb = it.block_tables, it.batch.max_blocks
    g = torch.Generator(device=it.device)
    g.manual_seed(rows)
    for _ in range(2):
        k, v = (torch.randint(-2 ** 15, 2 ** 15, (rows, n_kv_heads, head_dim), generator=g, device=it.device, dtype=torch.int16) for _ in "kv")
        got_k, got_v = torch.zeros_like(k), torch.zeros_like(v)
        B.cronus_kv_append(it.cache, k, v, cu, start, bt, mb, 4, rows)
        B.cronus_kv_gather(it.cache, got_k, got_v, cu, start, bt, mb, 4, rows)
        torch.cuda.synchronize()
        assert torch.equal(got_k, k) and torch.equal(got_v, v)
