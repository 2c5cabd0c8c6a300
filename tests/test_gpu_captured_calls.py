"""A captured cronus_attn_mixed call keeps its plan buffer, which the replays read.  The calls that
follow use the other buffers: more of them than the ring has must succeed, and replays in
between must give the bits of an eager call."""
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
    it.ensure_workspace()
    return batch, it


def call(batch, it):
    return B.cronus_attn_mixed(it.cache, it.q, it.out, batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks,
                               it.sm_scale, it.workspace, it.workspace_bytes, torch.cuda.current_stream().cuda_stream, check=False)


def test_calls_after_a_captured_one():
    batch, it = prepared([700, 3000, 9000, 40], [130, 1, 1, 1], seed=9600)
    other, it_other = prepared([900, 40, 2500], [1, 33, 1], seed=9601)
    for _ in range(9):  # every plan buffer of the ring exists before the capture
        assert call(batch, it) == B.CRONUS_OK and call(other, it_other) == B.CRONUS_OK
    torch.cuda.synchronize()
    want, want_other = bits_from_bf16_tensor(it.out).copy(), bits_from_bf16_tensor(it_other.out).copy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert call(batch, it) == B.CRONUS_OK
    for k in range(20):
        it_other.out.zero_()
        assert call(other, it_other) == B.CRONUS_OK, k
        it.out.zero_()
        if k % 3 == 0:
            graph.replay()
        else:
            assert call(batch, it) == B.CRONUS_OK, k
        torch.cuda.synchronize()
        assert np.array_equal(bits_from_bf16_tensor(it.out), want), k
        assert np.array_equal(bits_from_bf16_tensor(it_other.out), want_other), k
