"""The tuner's choice between a plan of the int8 kernels and the built-in one,
from the times per width.  No GPU call."""
from paper_2306_11006_amd import tune

BUILT_IN = [("split8", 16), ("tiles1", 256), ("kara2", 2**31 - 1)]
WINNERS = [(1, "split8"), (256, "tiles1"), (1024, "kara2")]
BEST = {"1": 2.8, "256": 7.3, "1024": 18.0}
TUNED = [("split8", 1), ("tiles1", 256), ("kara2", 2**31 - 1)]


def test_built_in_wins_where_it_is_faster():
    served = {"1": 2.2, "256": 2.7, "1024": 8.0}
    assert tune.pick_plan(WINNERS, BEST, served, BUILT_IN) == (BUILT_IN, served)


def test_kernels_win_where_they_are_faster():
    served = {"1": 2.9, "256": 7.2, "1024": 40.0}
    assert tune.pick_plan(WINNERS, BEST, served, BUILT_IN) == (TUNED, BEST)


def test_mixed_widths_go_by_the_geometric_mean():
    served = {"1": 2.2, "256": 2.7, "1024": 20.0}
    assert tune.pick_plan(WINNERS, BEST, served, BUILT_IN)[0] == BUILT_IN
    assert tune.pick_plan(WINNERS, BEST, dict(BEST), BUILT_IN)[0] == BUILT_IN


def test_without_the_transform_the_kernels_are_tuned():
    assert tune.pick_plan(WINNERS, BEST, {}, BUILT_IN) == (TUNED, BEST)
