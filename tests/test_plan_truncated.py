"""The planner's built-in rule for truncated cells with values above a lane's
column (host only), at its lines: values above the column, replicates of the
call, draws."""
import numpy as np
import pytest

from paper_1305_6738_amd import plan_forms


def above(alpha, n, K):
    w = np.arange(1, K + 1.0) ** -alpha
    return n * w[48:].sum() / w.sum()


@pytest.mark.parametrize("K,most", [(161, 64), (299, 64), (300, 84), (4096, 84)])
@pytest.mark.parametrize("alpha", [-0.5, 0.5, 1.0])
def test_values_above_the_column(K, most, alpha):
    n = int(most / above(alpha, 1, K))
    many = 10 ** 7
    assert plan_forms([(alpha, n, many, 1, 0, K)]) == ["lane"]
    assert plan_forms([(alpha, n + n // 10 + 1, many, 1, 0, K)])[0] != "lane"


@pytest.mark.parametrize("alpha,n,K", [(0.25, 20, 1000), (1.5, 500, 1000), (1.0, 98, 161)])
def test_replicates_of_the_call(alpha, n, K):
    a = above(alpha, n, K)
    R = int(np.ceil(80 * n + 710 / K ** 0.5 * a * a * a / n)) + 1
    assert plan_forms([(alpha, n, R, 1, 0, K)]) == ["lane"]
    assert plan_forms([(alpha, n, R - 2, 1, 0, K)]) == ["wave"]
    # the call's replicates count, not the cell's
    assert plan_forms([(alpha, n, R // 4 + 1, 1, i, K) for i in range(4)]) == ["lane"] * 4


def test_flat_laws_of_small_support_go_to_waves():
    # 50,000 replicates: 1,066 us by lanes, 657 by waves
    assert plan_forms([(-0.5, 100, 50000, 1, 0, 161)]) == ["wave"]


def test_eleven_draws():
    assert plan_forms([(1.0, n, 50000, 1, 0, 1000) for n in (10, 11, 15)]) == ["wave", "lane", "lane"]
