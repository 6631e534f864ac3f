"""Blocks of 64 tokens at head dim 128, lists of even length on one to two generations of workgroups: text rows and 64 lists per
XCD are cut where the call's lists are long, without counters.  Against the packed entry, which cuts nothing."""
import pytest

from test_gpu_small_blocks import _direct_twice_and_packed

pytestmark = pytest.mark.gpu


# just above one generation (1536 workgroups), in the middle, and grids beyond the rule's: more generations, lists too short
@pytest.mark.parametrize("blocks,heads,cut", [(121, 13, True), (118, 22, True), (121, 40, False), (62, 27, False)])
def test_lists_at_the_end_are_cut_where_they_are_long(blocks, heads, cut):
    vision, text = _direct_twice_and_packed(64, 128, blocks, heads, 0.3, False,
                                            lambda M: (0, 1, 2, M // 2, M - 1, M, M, M, M, M))
    assert (8 if cut else 0) <= int(vision.sum()) <= (512 if cut else 0)
    assert bool(text.any()) == cut
    vision, _ = _direct_twice_and_packed(64, 128, blocks, heads, 0.3, False, lambda M: (0, 1, 2, 3, 8))
    assert not vision.any()
