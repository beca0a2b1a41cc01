"""Truncated replicates with a short support in whole batches (16 lanes and
more walk the support themselves up to K = 100) and in small ones (a wave for
each): bit for bit the lane form's, and 32-bit counts against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


def run(ctx, cells, form):
    total = sum(c[2] for c in cells)
    D = torch.full((total,), float("nan"), dtype=torch.float64, device="cuda")
    A = torch.full_like(D, float("nan"))
    ctx.simulate_cells(cells, quantiles=None, form=form, d_out=D, alpha_hat_out=A)
    return D.cpu().numpy(), A.cpu().numpy()


@pytest.mark.parametrize("K", [17, 50, 66, 72, 99, 100, 101])
@pytest.mark.parametrize("alpha,n,R", [(0.25, 30, 60000), (1.5, 111, 60000), (4.0, 10, 3100)])
def test_batches_agree_with_the_lane_form(ctx, K, alpha, n, R):
    cells = [(alpha, n, R, 11, 2, K)]
    for x, y in zip(run(ctx, cells, "wave"), run(ctx, cells, "lane")):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("K", [20, 60, 100])
def test_wide_counts(ctx, orc, K):
    n, R = 70001, 40
    D, A = run(ctx, [(1.1, n, R, 3, 1, K)], "heavy")
    for rep in (0, R - 1):
        x = torch.zeros(n, dtype=torch.int64, device="cuda")
        f = torch.zeros(1, dtype=torch.int32, device="cuda")
        ctx.sample_draws(1.1, n, 3, 1, rep, 1, x, f, kmax=K)
        r = orc.tz_fit(x.cpu().numpy(), K)
        assert abs(A[rep] - r["alpha_hat"]) <= 1e-10 and abs(D[rep] - r["D"]) <= 1e-12
