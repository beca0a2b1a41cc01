"""The planner's built-in rule for long replicates of light tails (host only): a
lane takes as long for one as for many, so few of them go to a wave each, and
the lanes from 32 n replicates on, as measured."""
import pytest

from paper_1305_6738_amd import plan_forms


@pytest.mark.parametrize("n", [1001, 3000, 10000, 65535])
def test_few_long_replicates_of_the_pure_law(n):
    assert plan_forms([(3.5, n, 100, 1, 0)]) == ["wave"]
    assert plan_forms([(3.5, n, 32 * n - 1, 1, 0)]) == ["wave"]
    if n < 20000:  # (beyond, more than two values lie above a lane's column)
        assert plan_forms([(3.5, n, 32 * n, 1, 0)]) == ["lane"]


@pytest.mark.parametrize("n", [5001, 20000, 50000])
def test_few_long_replicates_of_a_short_support(n):
    assert plan_forms([(1.0, n, 333, 1, 0, 20)]) == ["wave"]
    assert plan_forms([(1.0, n, 32 * n, 1, 0, 20)]) == ["lane"]


def test_short_replicates_keep_the_lanes():
    assert plan_forms([(3.5, 1000, 100, 1, 0), (1.0, 5000, 100, 1, 1, 20)]) == ["lane", "lane"]
