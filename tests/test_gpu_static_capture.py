"""The entry point for callers that cannot allocate under HIP graph capture: its work list
travels in the captured launches' arguments (one launch, or several for a longer list), so a
replay needs nothing of the call that was captured.  Replays, with eager calls of another batch
and changed inputs in between, must give what an eager call gives."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu


def prepared(P, C, seed):
    batch = W.custom_batch(W.SHAPE_8B, P, C, seed=seed)
    it = DeviceIteration(batch, pool_fill=0)
    it.load_device_inputs()
    it.setup_decode_context()
    it.ingest_prefix()
    it.append_new()
    return batch, it


def call(batch, it):
    B.cronus_attn_mixed_static(it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables,
                               batch.max_blocks, it.sm_scale, torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("n", [5, 150])  # a list in one launch's arguments, and one that is uploaded in pieces
def test_replays_equal_eager_calls(n):
    rng = np.random.default_rng(n)
    batch, it = prepared(rng.integers(50, 3000, n).tolist() + [700], [1] * n + [130], seed=9200 + n)
    other, it_other = prepared([900, 40, 2500], [1, 33, 1], seed=9300 + n)
    call(batch, it)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(batch, it)
    for k in range(4):
        it.q.mul_(-1.5 if k % 2 else 0.75)
        call(other, it_other)
        call(batch, it)
        torch.cuda.synchronize()
        want = bits_from_bf16_tensor(it.out).copy()
        it.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), want)
        assert want.any()
