"""cronus_kv_append_pair leaves the bits of two cronus_kv_append calls: sets that meet inside a
block (the prefix ends, the new rows begin there), sequences without a row in one of the sets, an
empty set on either side, bf16 and fp8, D = 64 and 128."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration

pytestmark = pytest.mark.gpu

CASES = [
    (8, 128, "bf16", [0, 5, 16, 37, 1000, 3, 64], [9, 1, 20, 1, 333, 16, 7]),
    (2, 64, "fp8", [15, 17, 0, 100], [2, 1, 65, 31]),
    (8, 128, "fp8", [7, 250, 31], [1, 1, 1]),       # decodes only: the first set is empty
    (4, 64, "bf16", [0, 0, 0], [1, 40, 17]),        # whole prompts: the first set is empty
] + [(1, 128, "bf16", [3] * 130, [2] * 130)]        # more sequences than a wavefront's lanes


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("swap", [False, True])
def test_pair_equals_two_appends(case, swap):
    hkv, d, dt, P, C = CASES[case]
    batch = W.custom_batch(W.HeadShape(4 * hkv, hkv, d, dt), P, C, seed=60 + case)
    it = DeviceIteration(batch, pool_fill=0x5A)
    it.load_device_inputs()
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.ingest_prefix()
    it.append_new()
    want = it.k_pool.clone(), it.v_pool.clone()
    it.k_pool.fill_(0x5A)
    it.v_pool.fill_(0x5A)
    sets = [(it.prefix_k, it.prefix_v, it.cu_prefix, it.zero_pos, it.n_prefix_tokens),
            (it.new_k, it.new_v, it.cu_new, it.prefix_pos, it.n_new_tokens)]
    B.cronus_kv_append_pair(it.cache, *(sets[::-1] if swap else sets), it.block_tables, batch.max_blocks, batch.n_seqs,
                            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(it.k_pool, want[0]) and torch.equal(it.v_pool, want[1])
    assert np.any(want[0].cpu().numpy() != 0x5A)
