"""cronus_iteration leaves the bits of cronus_kv_append_pair followed by cronus_attn_mixed, in the cache and in the output: rows
that stay in the caches and rows stored past them (iterations bound by streaming, on either side of the rule), bf16 and fp8, D = 64
and 128, sets that meet inside a block, an empty set, sequences without rows, no query rows; blocks that another
sequence of the call reads; replays of a captured call; and refusals."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu

# streaming at 6 TB/s takes 20 us from 29 297 decode keys of 8 KV heads x 128 on
CASES = {
    "few decodes": (W.SHAPE_8B, [5, 16, 31, 700, 2999, 15], [1] * 6),
    "just below the rule": (W.SHAPE_8B, [9764, 9764, 9765], [1, 1, 1]),
    "just above the rule": (W.SHAPE_8B, [9764, 9765, 9765], [1, 1, 1]),
    "streaming, chunk and prefix": (W.SHAPE_8B, [1003, 20000, 20000], [37, 1, 1]),
    "streaming, fp8": (W.HeadShape(16, 8, 128, "fp8"), [250, 40000, 30000, 0], [70, 1, 1, 17]),
    "streaming, D 64": (W.HeadShape(8, 8, 64), [100, 60000, 17], [65, 1, 1]),
    "halves and edges": (W.SHAPE_8B, [3, 8, 24, 40, 0, 100], [5, 8, 16, 40, 1, 33]),
    "fp8, D 64": (W.HeadShape(8, 4, 64, "fp8"), [15, 17, 0, 100], [2, 1, 65, 31]),
    "fp8, bf16 copy": (W.HeadShape(16, 2, 64, "fp8"), [100, 40], [520, 1]),
    "whole prompts": (W.SHAPE_8B, [0, 0], [130, 47]),
    "skipped sequence": (W.SHAPE_8B, [50, 60, 70], [1, 0, 20]),
    "no query rows": (W.SHAPE_8B, [50, 60], [0, 0]),
    "shared blocks": (W.SHAPE_8B, [64, 70], [20, 1]),
}


def prepared(name):
    shape, P, C = CASES[name]
    it = DeviceIteration(W.custom_batch(shape, P, C, seed=77), pool_fill=0x5A)
    it.load_device_inputs()
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.setup_decode_context()
    it.ensure_workspace()
    return it


def fresh(it):
    it.k_pool.fill_(0x5A)
    it.v_pool.fill_(0x5A)
    it.out.zero_()
    it.setup_decode_context()


def state(it):
    torch.cuda.synchronize()
    return it.k_pool.clone(), it.v_pool.clone(), bits_from_bf16_tensor(it.out).copy()


def same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("name", CASES)
def test_iteration_equals_append_and_attention(name):
    it = prepared(name)
    if name == "shared blocks":  # the decode's first blocks are those that the chunk's prefix is placed in
        it.block_tables[1, :4] = it.block_tables[0, :4]
        fresh(it)
    if name == "fp8, bf16 copy":
        assert B.cronus_attn_mixed_plan_stats(it.cache, it.batch.prefix_lens, it.batch.chunk_lens)["copy_blocks"] > 0
    it.place_rows()
    it.attention()
    want = state(it)
    for _ in range(2):
        fresh(it)
        it.step()
        assert same(state(it), want)


def test_replays_and_refusals():
    it = prepared("streaming, chunk and prefix")
    it.step()
    want = state(it)
    b = it.batch
    call = lambda q, given: B.cronus_iteration(it.cache, *it._rows(), q, it.out, b.prefix_lens, b.chunk_lens, it.block_tables,
                                               b.max_blocks, it.sm_scale, it.workspace, given, it._stream(), check=False)
    fresh(it)
    before = state(it)
    assert call(None, it.workspace_bytes) == B.CRONUS_ERR_INVALID_ARG and same(state(it), before)
    # refused on the host, with nothing enqueued: a sequence longer than its row of the table, no workspace
    long = b.prefix_lens.copy()
    long[-1] = 16 * b.max_blocks
    for P, ws, code in ((long, it.workspace, B.CRONUS_ERR_INVALID_ARG), (b.prefix_lens, None, B.CRONUS_ERR_WORKSPACE)):
        assert B.cronus_iteration(it.cache, *it._rows(), it.q, it.out, P, b.chunk_lens, it.block_tables, b.max_blocks, it.sm_scale, ws,
                                  it.workspace_bytes, it._stream(), check=False) == code
        assert same(state(it), before)
    assert call(it.q, 256) == B.CRONUS_ERR_WORKSPACE  # found when the plan is built: the rows are there, the output is not
    got = state(it)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and np.array_equal(got[2], before[2])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        it.step()
    for k in range(4):
        fresh(it)
        torch.cuda.synchronize()
        graph.replay()
        assert same(state(it), want), k


@pytest.mark.parametrize("device", ["cuda:0", "cuda"])
def test_a_step_runs_on_the_current_stream(device):
    shape, P, C = CASES["halves and edges"]
    it = DeviceIteration(W.custom_batch(shape, P, C, seed=77), device=device, pool_fill=0x5A)
    it.load_device_inputs()
    it.setup_decode_context()
    it.step()
    want = state(it)
    assert it._stream() == torch.cuda.current_stream(it.device).cuda_stream
    side = torch.cuda.Stream()
    fresh(it)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        assert it._stream() == side.cuda_stream
        it.step()
        done = torch.cuda.Event()
        done.record()
    assert it._stream() == torch.cuda.current_stream(it.device).cuda_stream
    torch.cuda.current_stream().wait_event(done)
    assert same(state(it), want)
