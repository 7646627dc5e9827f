"""Which call sequence a step takes by itself: forward and sort in one launch, or the next batch's sort beside this batch's
step.  The shapes are those at which the two were timed (microseconds in ``step_sequence``)."""
import pytest

from paper_2103_00686_amd.hotpath import step_sequence


def _auto(nt, n, rows, dim, **kw):
    return step_sequence([rows] * nt, dim, True, n, nt * n, **kw)


@pytest.mark.parametrize("nt,n,rows,dim", [(8, 100_000, 40, 16), (8, 100_000, 1000, 16), (8, 100_000, 8000, 16), (8, 100_000, 30_000, 16),
                                           (13, 65_536, 40, 16), (13, 65_536, 8000, 16), (26, 30_000, 40, 16), (20, 50_000, 255, 32),
                                           (16, 100_000, 200, 16), (10, 100_000, 1000, 32), (13, 60_000, 1000, 16), (13, 100_000, 65_000, 16)])
def test_long_lists_on_few_slots_are_sorted_ahead(nt, n, rows, dim):
    """One launch took up to 1.3 times as long there."""
    assert _auto(nt, n, rows, dim) == "ahead"
    assert _auto(nt, n, rows, dim, single_stream=True) == "fused"


@pytest.mark.parametrize("nt,n,rows,dim", [(1, 1024, 40, 16), (26, 16_384, 40, 16), (8, 60_000, 40, 16), (1, 100_000, 40, 16), (8, 100_000, 40, 64),
                                           (26, 50_001, 400_000, 64), (8, 100_000, 65_536, 16), (13, 65_536, 30_000, 16), (26, 60_000, 1000, 16),
                                           (26, 100_000, 40, 16), (13, 50_000, 8000, 16), (20, 100_000, 8000, 16), (4, 100_000, 1000, 16)])
def test_other_one_hot_steps_are_one_launch(nt, n, rows, dim):
    assert _auto(nt, n, rows, dim) == "fused"


def test_bags_and_longer_batches():
    assert _auto(1, 100_001, 1_000_000, 16) == "ahead"
    assert _auto(26, 262_144, 1_000_000, 16) == "fused"  # beyond 4 M lookups
    assert step_sequence([10], 16, False, 2048, 102_400) == "ahead"
    assert step_sequence([10], 16, False, 2048, 102_400, single_stream=True) == "fused"
