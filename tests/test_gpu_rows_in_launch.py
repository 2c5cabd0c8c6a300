"""Decode iterations place their rows in the attention launch (one set with a row for each of at most 64 decodes): the bits
of cronus_kv_append followed by cronus_attn_mixed, in the cache and in the output, on either side of that rule (SCATTERED: the cases
beyond it, which tests/test_iteration_route_cpu.py checks).  Rows one a
sequence in order, and, since the counts are on the device, otherwise: several or none of a sequence, rows past its length or of a sequence
without query rows (no item reads them), rows that other sequences read too, at the first and last slot of a block, in spans that are not the
last, more (row, KV head) pairs than work-groups.  Beyond the rule also: rows that stay whole, for which table entries are loaded more than once."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu

G4, G7, D64, MQA = W.SHAPE_8B, W.HeadShape(28, 4, 128), W.HeadShape(8, 2, 64), W.HeadShape(48, 1, 128)
FP8, FP8_64 = W.HeadShape(16, 8, 128, "fp8"), W.HeadShape(8, 4, 64, "fp8")

# shape, cached keys and query rows of the sequences, rows placed (count of each sequence, first position; None: its new row)
CASES = {
    "one key": (G4, [0], [1], None),
    "slots": (G4, [15, 16, 31, 32, 255, 256, 511], [1] * 7, None),
    "64": (G4, list(range(64)), [1] * 64, None),
    "65": (G4, list(range(65)), [1] * 65, None),
    "spans": (G7, [5000, 900, 9000], [1] * 3, None),
    "fp8": (FP8, [5000, 900, 17, 31], [1] * 4, None),
    "fp8, D 64": (FP8_64, list(range(40, 100)), [1] * 60, None),
    "D 64": (D64, [700, 63, 64], [1] * 3, None),
    "two head groups": (MQA, [700, 31], [1, 1], None),
    "few work-groups": (W.HeadShape(64, 64, 64), [3] * 64, [0] * 63 + [1], ([1] * 64, [3] * 64)),
    "short chunks": (G4, [100, 30, 7], [8, 1, 5], ([8, 1, 5], [100, 30, 7])),
    "some without rows": (G4, [100, 600, 40], [1, 1, 1], ([0, 1, 0], [100, 600, 40])),
    "rows in other spans": (G4, [3000, 600], [1, 1], ([20, 7], [1015, 250])),
    "rows past the length": (G4, [100, 600, 40, 80], [1, 1, 0, 1], ([3, 2, 9, 1], [120, 601, 33, 0])),
    "fp8, rows past the length": (FP8, [100, 600, 40], [1, 0, 1], ([5, 11, 1], [99, 590, 40])),
    "read by others": (G4, [40, 41, 42, 600], [1] * 4, "shared"),
    "read by others, fp8": (FP8, [40, 41, 42, 600], [1] * 4, "shared"),
    "left whole": (W.HeadShape(1040, 1040, 64), [8250, 8210, 8195, 8400], [1] * 4, ([1, 30, 1, 1], [8250, 8190, 8195, 100])),
    # as many rows as decodes, but not one of each
    "of one sequence": (G4, [100] * 20, [1] * 20, ([20] + [0] * 19, [77] + [100] * 19)),
    "of one sequence, D 64": (D64, [900, 40, 600], [1] * 3, ([0, 3, 0], [900, 38, 600])),
    "out of order": (G4, [100, 30, 7, 900], [1] * 4, ([1, 0, 2, 1], [100, 30, 6, 900])),
    "in other spans": (G7, [3000, 600] + [50] * 25, [1] * 27, ([20, 7] + [0] * 25, [1015, 250] + [0] * 25)),
    "past the length": (G4, [100, 600, 40, 80] + [33] * 11, [1] * 15, ([3, 2, 9, 1] + [0] * 11, [120, 601, 33, 0] + [0] * 11)),
    "fp8, past the length": (FP8, [100, 600, 40] + [17] * 14, [1] * 17, ([5, 11, 1] + [0] * 14, [99, 590, 45] + [0] * 14)),
    "skipped among 8": (G7, [100, 600, 15, 40, 2100, 31, 16, 5], [1, 0, 1, 1, 1, 0, 0, 1], ([1, 0, 1, 1, 1, 0, 0, 1], [100, 600, 15, 40, 2100, 31, 16, 5])),
    "fp8, skipped among 3": (FP8, [100, 600, 15], [0, 1, 0], ([0, 1, 0], [100, 600, 15])),
    "skipped among 9": (G4, [100, 600, 15, 40, 900, 31, 16, 5, 8], [1] * 8 + [0], ([1] * 8 + [0], [100, 600, 15, 40, 900, 31, 16, 5, 8])),
    "fewer rows than counted": (G4, [100, 600, 40], [1] * 3, ([1, 1, 0], [100, 600, 40])),
    "more heads than work-groups": (W.HeadShape(1040, 1040, 64), [100], [1], ([1], [120])),
}
SCATTERED = ("65", "few work-groups", "short chunks", "some without rows", "rows in other spans", "rows past the length", "fp8, rows past the length",
             "left whole", "skipped among 9", "fewer rows than counted")


@pytest.mark.parametrize("name", CASES)
def test_rows_placed_in_the_launch(name):
    shape, P, C, given = CASES[name]
    n = len(P)
    shared = given == "shared"
    counts, starts = (C, P) if given is None or shared else given
    # tables with room for the rows past a sequence's length
    it = DeviceIteration(W.custom_batch(shape, [p + 48 for p in P], [max(c, 1) for c in C], seed=91), pool_fill=0)
    if shared:  # sequences 1 and 2 continue sequence 0: each reads the rows before its own; 3 has them in a block of its middle
        it.block_tables[1:3, :6] = it.block_tables[0, :6]
        it.block_tables[3, 20] = it.block_tables[0, 2]
    sh = it.batch.shape
    g = torch.Generator(device=it.device)
    g.manual_seed(5)
    mk = lambda *s: (torch.randn(s, generator=g, device=it.device) * 0.125).to(torch.bfloat16)
    if it.fp8:
        it.set_fp8_scales(np.full(sh.n_kv_heads, 0.5 / 448, np.float32), np.full(sh.n_kv_heads, 0.75 / 448, np.float32))
        pools = [torch.randint(0, 0x60, p.shape, generator=g, device=it.device, dtype=torch.uint8) for p in (it.k_pool, it.v_pool)]
    else:
        pools = [torch.randint(0x3c00, 0x3e00, p.shape, generator=g, device=it.device, dtype=torch.int16) for p in (it.k_pool, it.v_pool)]
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=it.device)
    rows = int(sum(counts))
    k, v, q = mk(rows, sh.n_kv_heads, sh.head_dim), mk(rows, sh.n_kv_heads, sh.head_dim), mk(sum(C), sh.n_q_heads, sh.head_dim)
    cu, start = i32([0] + list(np.cumsum(counts))), i32(starts)
    out = torch.empty_like(q)
    ws = torch.empty(B.cronus_attn_mixed_workspace_bytes(it.cache, P, C), dtype=torch.uint8, device=it.device)
    some, none = (k, v, cu, start, rows), (None, None, None, None, 0)
    bt, mb = it.block_tables, it.batch.max_blocks

    def run(f):
        it.k_pool.copy_(pools[0])
        it.v_pool.copy_(pools[1])
        out.fill_(float("nan"))
        f()
        torch.cuda.synchronize()
        return it.k_pool.clone(), it.v_pool.clone(), bits_from_bf16_tensor(out).copy()

    def two_calls():
        B.cronus_kv_append(it.cache, k, v, cu, start, bt, mb, n, rows)
        B.cronus_attn_mixed(it.cache, q, out, P, C, bt, mb, it.sm_scale, ws, ws.numel())

    one_call = lambda a, b: lambda: B.cronus_iteration(it.cache, a, b, q, out, P, C, bt, mb, it.sm_scale, ws, ws.numel())
    want = run(two_calls)
    assert not torch.equal(want[0], pools[0])
    for a, b in ((some, none), (none, some), (some, none)):
        got = run(one_call(a, b))
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert np.array_equal(got[2], want[2])
    if name == "left whole":
        items = B.cronus_attn_mixed_plan_items(it.cache, P, C)
        assert (items[:, 7] - items[:, 6]).max() > 32 * 256  # a wave's 32 sub-tiles, for which it loads entries at once
    if name in ("spans", "left whole"):
        # a workspace that is too small: the rows are there, the output is not
        assert B.cronus_attn_mixed_plan_stats(it.cache, P, C)["partials"] > 0
        got = run(lambda: B.cronus_iteration(it.cache, some, none, q, out, P, C, bt, mb, it.sm_scale, ws, 256, check=False))
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and (got[2] & 0x7fff == 0x7fc0).all()
    if name in ("spans", "past the length"):
        run(one_call(some, none))
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                B.cronus_iteration(it.cache, some, none, q, out, P, C, bt, mb, it.sm_scale, ws, ws.numel(), stream.cuda_stream)
        for _ in range(3):
            got = run(graph.replay)
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and np.array_equal(got[2], want[2])


@pytest.mark.parametrize("where", ["out", "workspace"])
def test_rows_that_lie_in_what_the_attention_writes(where):
    """As with the two calls, the rows and their counts may lie in the output or in the workspace: they are read first."""
    shape, P = G4, [5000, 900, 17, 31, 2000, 3100, 255, 256]
    n, C = len(P), [1] * len(P)
    it = DeviceIteration(W.custom_batch(shape, P, C, seed=92), pool_fill=0)
    it.load_device_inputs()
    it.setup_decode_context()
    pools = it.k_pool.clone(), it.v_pool.clone()
    ws = torch.zeros(B.cronus_attn_mixed_workspace_bytes(it.cache, P, C) + (1 << 20), dtype=torch.uint8, device=it.device)
    out = torch.zeros_like(it.q)
    area = (out if where == "out" else ws).view(torch.uint8).reshape(-1)
    arrays, at = [], 0
    for a in (it.new_k, it.new_v, it.cu_new, it.prefix_pos):
        size = a.numel() * a.element_size()
        arrays.append((a, area[at:at + size].view(a.dtype).reshape(a.shape)))
        at += (size + 15) // 16 * 16
    assert at <= area.numel()

    def run(f):
        it.k_pool.copy_(pools[0])
        it.v_pool.copy_(pools[1])
        for a, moved in arrays:
            moved.copy_(a)
        f(*(moved for _, moved in arrays))
        torch.cuda.synchronize()
        return it.k_pool.clone(), it.v_pool.clone(), bits_from_bf16_tensor(out).copy()

    def two_calls(k, v, cu, start):
        B.cronus_kv_append(it.cache, k, v, cu, start, it.block_tables, it.batch.max_blocks, n, n)
        B.cronus_attn_mixed(it.cache, it.q, out, P, C, it.block_tables, it.batch.max_blocks, it.sm_scale, ws, ws.numel())

    def one_call(k, v, cu, start):
        B.cronus_iteration(it.cache, (k, v, cu, start, n), (None, None, None, None, 0), it.q, out, P, C, it.block_tables, it.batch.max_blocks,
                           it.sm_scale, ws, ws.numel())

    want = run(two_calls)
    for _ in range(3):
        got = run(one_call)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and np.array_equal(got[2], want[2])
