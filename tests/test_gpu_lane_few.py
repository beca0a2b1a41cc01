"""The lane form's finish with few values above a lane's column (up to 12 in
every lane of the wave: one bucket) and with more (buckets): bit for bit the
wave form's, and sampled replicates against the oracle (alpha_hat 1e-10, D
1e-12).  At alpha = 1.05 nearly every draw is above the column of 48."""
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


def run(ctx, cell, form):
    D = torch.full((cell[2],), float("nan"), dtype=torch.float64, device="cuda")
    A = torch.full_like(D, float("nan"))
    FP = torch.zeros(cell[2], dtype=torch.int64, device="cuda")
    ctx.simulate_cells([cell], quantiles=None, form=form, d_out=D, alpha_hat_out=A,
                       fingerprint_out=FP)
    return D.cpu().numpy(), A.cpu().numpy(), FP.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n", [1, 2, 11, 12, 13, 14, 20, 60])
@pytest.mark.parametrize("alpha,K", [(1.05, 0), (1.5, 0), (3.0, 0), (0.2, 4096), (1.5, 161)])
def test_few_values(ctx, orc, alpha, K, n):
    R = 330
    lane, wave = run(ctx, (alpha, n, R, 17, 4, K), "lane"), run(ctx, (alpha, n, R, 17, 4, K), "wave")
    for x, y in zip(lane, wave):
        assert np.array_equal(x, y)
    if K == 0:
        r = orc.simulate(alpha, n, 17, 4, 0, R)
        assert np.array_equal(lane[2], r["fp"])
        assert np.max(np.abs(lane[1] - r["alpha_hat"]) / r["alpha_hat"]) < 1e-10
        assert np.max(np.abs(lane[0] - r["D"])) < 1e-12
