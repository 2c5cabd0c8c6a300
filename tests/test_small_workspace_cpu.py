"""A workspace that holds what the library asked for these lengths before it cut chunk tiles into finer
spans (versions up to 505; the sizes below are theirs) is accepted, one byte less is not.  Without a GPU a
call whose workspace is accepted ends with the HIP error of the set-up, before anything is launched."""
import pytest
import torch

from paper_2509_17357_amd import binding as B

BF16, FP8 = B.CRONUS_KV_BF16, B.CRONUS_KV_FP8_E4M3
# (heads, cache, prefixes, chunks, bytes up to version 505); the last two need no more now
CASES = [((32, 8, 128), BF16, [0], [1200], 256), ((32, 8, 128), FP8, [1100], [400], 256),
         ((28, 4, 128), BF16, [1800, 2500], [300, 1], 9917440), ((8, 2, 64), BF16, [900, 4000], [700, 1], 135168),
         ((64, 8, 128), FP8, [1500, 2500], [100, 1], 7454720), ((32, 8, 128), BF16, [2500, 2500, 7000], [200, 1, 1], 12912640),
         ((32, 8, 128), BF16, [0], [700], 256), ((64, 8, 128), FP8, [4000, 2500, 700], [200, 1, 90], 23029760)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where nothing can be launched")
@pytest.mark.parametrize("heads, dtype, P, C, before", CASES)
def test_workspace_of_earlier_versions_is_accepted(heads, dtype, P, C, before):
    fake = 0x7F0000001000
    scale = fake if dtype == FP8 else None
    cache = B.make_cache(fake, fake, 1 << 20, *heads, k_scale=scale, v_scale=scale, kv_dtype=dtype)
    call = lambda n: B.cronus_attn_mixed(cache, fake, fake, P, C, fake, 1024, 0.1, fake, n, check=False)
    need = B.cronus_attn_mixed_workspace_bytes(cache, P, C)
    assert call(need) == B.CRONUS_ERR_HIP
    least = min(need, before)
    assert call(least) == B.CRONUS_ERR_HIP
    assert call(least - 1) == B.CRONUS_ERR_WORKSPACE
    assert (need > before) == (CASES.index((heads, dtype, P, C, before)) < 6)
