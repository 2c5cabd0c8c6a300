"""Calls whose workspace is smaller than the present need but holds that of versions up to 505: the
coarser cut stays inside it and matches the oracle, and the next call with the full workspace is that
of a first one."""
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import bits_from_bf16_tensor

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [((32, 8, 128, "bf16"), [0], [1200], 256), ((32, 8, 128, "fp8"), [1100], [400], 256),
         ((28, 4, 128, "bf16"), [1800, 2500], [300, 1], 9917440), ((64, 8, 128, "fp8"), [1500, 2500], [100, 1], 7454720)]
GUARD = 1 << 20


@pytest.mark.parametrize("heads, P, C, size", CASES)
def test_smaller_workspace_matches_the_oracle(heads, P, C, size):
    batch = W.custom_batch(W.HeadShape(*heads), P, C, seed=77)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    q = batch.gen_q()
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    assert it.workspace_bytes > size
    ws = torch.full((size + GUARD,), 0x5A, dtype=torch.uint8, device=it.device)
    assert ws.data_ptr() % 256 == 0
    it.out.zero_()
    args = (it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks, it.sm_scale)
    B.cronus_attn_mixed(*args, ws, size, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((ws[size:] == 0x5A).all())
    U.check_rows_by_sequence(batch, bits_from_bf16_tensor(it.out), q, lambda s: kv[s], it.sm_scale, ks, vs)
    it.attention()
    torch.cuda.synchronize()
    assert (bits_from_bf16_tensor(it.out) == out).all()
