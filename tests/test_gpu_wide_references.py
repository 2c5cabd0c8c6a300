"""Wide tiles whose scores climb: the running reference of a row has to follow where a score
outgrows it, in the steady-state loop (which learns it from the numerators, two row tiles at
different times) and in the steps around it.  Ramps just under and just over the slack of 8 bits
a sub-tile, of many bits, and past the range of fp32; rows that see the same keys fall; contexts of one
to many sub-tiles; rows that end inside a wave's 16-row tile."""
import numpy as np
import pytest

from paper_2509_17357_amd import workloads as W

import parity_util as U

pytestmark = pytest.mark.gpu

SHAPES = [(32, 8, 128, "bf16"), (8, 2, 64, "bf16"), (28, 4, 128, "bf16"), (16, 2, 128, "fp8"), (8, 4, 64, "fp8")]
BITS_PER_SUBTILE = [7.5, 8.5, 40.0, 300.0]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("bits", BITS_PER_SUBTILE)
def test_reference_follows_climbing_scores(shape, bits):
    hq, hkv, d, dt = SHAPES[shape]
    C = [9, 70, 131, 64, 37, 200]
    P = [0, 0, 5, 700, 1023, 190]
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=910 + shape)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    scale = 1.0 / np.sqrt(d)
    # q = +-1 in the first dim, k there a ramp: score in bits = scale * log2(e) * q * k
    step = bits / (scale * 1.4426950408889634)
    for s, (k, v) in enumerate(kv):
        ramp = np.repeat(np.arange((k.shape[0] + 31) // 32), 32)[:k.shape[0]] * step
        k[:, :, 0] = W.f32_to_bf16_bits(ramp.astype(np.float32))[:, None]
    q = batch.gen_q()
    sign = np.where(np.arange(hq) % 3 == 2, -1.0, 1.0).astype(np.float32)
    q[:, :, 0] = W.f32_to_bf16_bits(sign)[None, :]
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)
