"""Q and output rows at addresses that are not multiples of 16 bytes (bf16 views with an offset
of one element, or of four): the results are the bits that aligned rows give.  Chunk tiles first
of a work-group and reserved ahead, tiles whose rows end inside a wave's share, decodes, key
spans, both cache types and head sizes, both entry points."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bits_from_bf16_tensor

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, kv_dtype, prefix_lens, chunk_lens)
    (32, 8, 128, "bf16", [300, 4000, 70, 900], [100, 1, 33, 1]),
    (28, 4, 128, "bf16", [0] * 40 + [2000], list(range(300, 700, 10)) + [1]),  # tiles are reserved ahead
    (8, 2, 64, "bf16", [500, 1200], [70, 1]),
    (64, 8, 128, "fp8", [9000, 500, 40], [90, 1, 31]),
    (16, 2, 128, "fp8", [100, 3000], [530, 1]),                               # tiles that read the bf16 copy
    (8, 2, 64, "fp8", [3000, 700], [100, 1]),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_rows_at_any_address(case):
    hq, hkv, d, dt, P, C = CASES[case]
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=8800 + case)
    it = DeviceIteration(batch, pool_fill=0)
    it.load_device_inputs()
    if it.fp8:
        it.set_fp8_scales(*it.amax_scales())
    it.setup_decode_context()
    it.step()
    stream = torch.cuda.current_stream().cuda_stream
    lens = (batch.prefix_lens, batch.chunk_lens, it.block_tables, batch.max_blocks, it.sm_scale)
    calls = {"workspace": lambda q, out: B.cronus_attn_mixed(it.cache, q, out, *lens, it.workspace, it.workspace.numel(), stream),
             "static": lambda q, out: B.cronus_attn_mixed_static(it.cache, q, out, *lens, stream)}
    for name, call in calls.items():
        call(it.q, it.out)
        torch.cuda.synchronize()
        want = bits_from_bf16_tensor(it.out).copy()
        assert want.any()
        for off_q, off_out in [(1, 0), (0, 1), (4, 4), (7, 3)]:
            view = lambda off: torch.zeros(it.q.numel() + 16, dtype=torch.bfloat16, device=it.q.device)[off:off + it.q.numel()]
            q, out = view(off_q).view(it.q.shape), view(off_out).view(it.q.shape)
            q.copy_(it.q)
            assert q.data_ptr() % 16 == 2 * off_q and out.data_ptr() % 16 == 2 * off_out
            call(q, out)
            torch.cuda.synchronize()
            assert np.array_equal(bits_from_bf16_tensor(out), want), (name, off_q, off_out)
