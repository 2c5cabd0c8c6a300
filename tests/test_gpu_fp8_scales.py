"""Quantise-on-append under scales on both sides of the range in which quotients come from a
reciprocal and a residual (2^-64 .. 2^64) and far outside, odd mantissas among them: the codes of all
finite bf16 inputs (zeros of both signs and subnormals too) equal the software quantiser's; infinities and
NaNs get the same codes on both sides."""
import numpy as np
import pytest
import torch

from paper_2509_17357_amd import binding as B
from paper_2509_17357_amd import workloads as W
from paper_2509_17357_amd.runtime import DeviceIteration, bf16_tensor_from_bits

import parity_util as U

pytestmark = pytest.mark.gpu

D, HKV = 128, 8
EDGE = [2.0 ** -64, float(np.nextafter(np.float32(2.0 ** -64), np.float32(0))), 2.0 ** 64,
        float(np.nextafter(np.float32(2.0 ** 64), np.float32(np.inf))), 2.0 ** -100, 2.0 ** 100, 2.0 ** -126, 3e38]
SCALES = [EDGE, [float(2.0 ** e * m) for e, m in zip(range(-62, 64, 16), (1.1, 1.9999999, 1.3333334, 1.0000001, 1.5, 1.7, 1.25, 1.99))],
          np.random.default_rng(5).uniform(1e-6, 1e-1, 8).tolist()]


def run(values, scales):
    n_tok = values.size // D
    src = np.repeat(values.reshape(n_tok, 1, D), HKV, axis=1)
    batch = W.custom_batch(W.HeadShape(HKV, HKV, D, "fp8"), [0], [n_tok], seed=5401)
    it = DeviceIteration(batch, pool_fill=0x7F)
    ks = np.array(scales, dtype=np.float32)
    it.set_fp8_scales(ks, ks)
    it.new_k = it.new_v = bf16_tensor_from_bits(src, it.device)
    it.append_new()
    torch.cuda.synchronize()
    return batch, src, ks, it


@pytest.mark.parametrize("group", range(len(SCALES)))
def test_codes_of_every_finite_input(group):
    vals = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    finite = vals[((vals >> 7) & 0xFF) != 0xFF]
    batch, src, ks, it = run(finite, SCALES[group])
    kp, vp = U.oracle_pools(batch, [(src, src)], fill=0x7F, k_scale=ks, v_scale=ks)
    assert np.array_equal(it.k_pool.cpu().numpy(), kp)
    assert np.array_equal(it.v_pool.cpu().numpy(), vp)


def test_codes_of_infinities_and_nans():
    vals = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    other = vals[((vals >> 7) & 0xFF) == 0xFF]
    batch, src, ks, it = run(other, EDGE)
    n = src.shape[0]
    rows = [torch.zeros((n, HKV, D), dtype=torch.uint8, device=it.device) for _ in range(2)]
    B.cronus_kv_gather(it.cache, *rows, it.cu_new, it.zero_pos, it.block_tables, batch.max_blocks, 1, n,
                       torch.cuda.current_stream().cuda_stream)
    for got in rows:
        got = got.cpu().numpy()
        assert (got == got[:, 4:5, :]).all()        # head 4 (scale 2^-100) divides, heads 0 and 2 do not
        inf = (other.reshape(n, D) & 0x7F) == 0
        assert (got[:, 0, :][inf] & 0x7F == 0x7E).all()   # 448
