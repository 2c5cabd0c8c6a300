"""Wide tiles whose scores climb: the running reference of a row has to follow where a score
outgrows it, in the steady-state loop (which learns it from the numerators) and in the steps around it.
Ramps just under and just over the slack of 8 bits a sub-tile (on a bf16 cache: fp8 codes round the ramp to
steps of several sub-tiles), of many bits, and past the range of fp32; rows that see the same keys fall; contexts of one
to many sub-tiles; rows that end inside a wave's 16-row tile.  Then rows that climb in one of a wave's two 16-row
tiles only, down to a single one, and single keys at each of the 32 places of a sub-tile: every packed numerator of either
tile alone has to send the step to the rescaling, or 300 bits overflow."""
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


# rows of a wave's 32 that see the ramp climb (the others see it fall); row = token of the tile x heads + head
ROWS = [range(16), range(16, 32), [0], [13], [15], [16], [22], [31]]


def signs(shape, C, rows):
    """+-1 by query row and head, [sum(C), heads]: + where the row's place in its wave is in `rows`."""
    hq, hkv = shape[:2]
    g = hq // hkv
    tok = 256 // g
    out = []
    for c in C:
        t, h = np.meshgrid(np.arange(c) % tok, np.arange(hq) % g, indexing="ij")
        out.append(np.where(np.isin((t * g + h) % 32, list(rows)), 1.0, -1.0))
    return np.concatenate(out).astype(np.float32)


def run(shape, C, P, seed, k0_of, rows):
    """Batch whose keys have k0_of(sequence, length) in dim 0 and whose query rows have +-1 there."""
    hq, hkv, d, dt = shape
    batch = W.custom_batch(W.HeadShape(hq, hkv, d, dt), P, C, seed=seed)
    kv = [batch.gen_kv(s) for s in range(batch.n_seqs)]
    for s, (k, v) in enumerate(kv):
        k[:, :, 0] = W.f32_to_bf16_bits(k0_of(s, k.shape[0]).astype(np.float32))[:, None]
    q = batch.gen_q()
    q[:, :, 0] = W.f32_to_bf16_bits(signs(shape, C, rows))
    out, ks, vs, it = U.run_hot_path(batch, q, kv)
    U.check_rows_by_sequence(batch, out, q, lambda s: kv[s], it.sm_scale, ks, vs)


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("rows", range(len(ROWS)))
def test_one_row_tile_climbs(shape, rows):
    hq, hkv, d, dt = SHAPES[shape]
    step = 300.0 * np.sqrt(d) / 1.4426950408889634
    ramp = lambda s, n: np.repeat(np.arange((n + 31) // 32), 32)[:n] * step
    run(SHAPES[shape], [64, 37, 130], [480, 511, 0], 930 + shape, ramp, ROWS[rows])


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("sub", [4, 5])
def test_single_keys_at_every_place_of_a_sub_tile(shape, half, sub):
    d = SHAPES[shape][2]
    high = 300.0 * np.sqrt(d) / 1.4426950408889634

    def k0(s, n):  # sequence s: key s of sub-tile `sub`, which the steady loop takes
        k = np.zeros(n)
        k[32 * sub + s] = high
        return k
    run(SHAPES[shape], [18] * 32, [400 + 3 * s for s in range(32)], 940 + shape, k0, ROWS[half])
