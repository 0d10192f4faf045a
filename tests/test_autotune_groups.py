"""The autotuner's choice among XCD groups that may be one and the same launch."""
from paper_2206_15117_amd import autotune


def test_equal_launches_give_the_smallest_group():
    assert autotune.best_group({1: 21.00, 2: 18.10, 4: 18.07, 8: 18.09, 16: 18.06, 32: 18.11}) == 2
    assert autotune.best_group({1: 5.00, 2: 4.90, 4: 4.80, 8: 5.10}) == 4
    assert autotune.best_group({1: 3.0}) == 1
