"""Whole prompts and chunks with little context whose tiles differ in length: a little more than a round of
them is not cut into key spans (measured, attention of the launch uncut and in the least cut, us: 40.0 / 51.6,
39.4 / 49.0, 42.8 / 52.3, 43.5 / 52.1, 58.5 / 66.6, 55.8 / 62.2), where tiles of nearly one length, which
would need a second whole round, still are."""
import pytest

from paper_2509_17357_amd import workloads as W

from test_plan_cpu import plan_for


@pytest.mark.parametrize("heads, P, C, tiles", [((64, 8, 128), [0], [1228], 312), ((28, 4, 128), [0, 0], [1174, 1356], 284),
                                                ((28, 4, 128), [0, 0, 0], [742, 1149, 1178], 344),
                                                ((32, 8, 128), [0, 0, 0], [742, 1149, 1178], 392),
                                                ((32, 8, 128), [686, 529, 970], [821, 811, 815], 312),
                                                ((28, 4, 128), [259, 0, 101], [1916, 502, 619], 344)])
def test_tiles_of_many_lengths_stay_whole(heads, P, C, tiles):
    _, stats = plan_for(W.HeadShape(*heads), P, C)
    assert stats["wide_items"] == tiles


@pytest.mark.parametrize("heads, P, C, uncut", [((32, 8, 128), [16384], [496], 64), ((64, 8, 128), [4620], [1112], 280)])
def test_tiles_of_one_length_are_cut(heads, P, C, uncut):
    _, stats = plan_for(W.HeadShape(*heads), P, C)
    assert stats["wide_items"] >= 2 * uncut
