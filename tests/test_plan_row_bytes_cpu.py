"""Wide tiles address their rows by 24-bit products of the bytes of a token's heads: a token of
2^24 bytes or more must not get one, and is covered by narrow items all the same."""
import numpy as np
import pytest

from paper_2509_17357_amd import workloads as W

from test_plan_cpu import F, check_plan


@pytest.mark.parametrize("hq, hkv, d, chunk, wide", [
    (65472, 1, 128, 2, True), (65536, 1, 128, 2, False), (70000, 2, 128, 2, False), (131072, 4, 64, 2, False), (131008, 4, 64, 2, True),
    (65536, 65536, 128, 33, False)])
def test_tiles_of_very_many_heads(hq, hkv, d, chunk, wide):
    if hkv > 4:  # too many heads to walk: the kinds of items only
        from test_plan_cpu import plan_for
        items, _ = plan_for(W.HeadShape(hq, hkv, d), [5], [chunk])
    else:
        items, _ = check_plan(W.HeadShape(hq, hkv, d), [300], [chunk])
    assert ((items[:, F["wide"]] >= 1).any()) == wide
    rows = items[:, F["n_tok"]] * items[:, F["n_heads"]]
    assert rows.sum() == hq * chunk
