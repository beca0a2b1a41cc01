"""GPU parity of the truncated law in the lane form with many values above a
lane's column: from the K that takes Euler-Maclaurin sums on, at the edges of
the column (48 values), of the line that chooses the form, and with more
values than a lane keeps (escalated).  The forms agree bit for bit, and with the
oracle as everywhere (alpha_hat 1e-10, D 1e-12, flags equal)."""
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
    D = torch.zeros(total, dtype=torch.float64, device="cuda")
    A = torch.zeros_like(D)
    F = torch.zeros(total, dtype=torch.int32, device="cuda")
    ctx.simulate_cells(cells, quantiles=None, form=form, d_out=D, alpha_hat_out=A, flags_out=F)
    return D.cpu().numpy(), A.cpu().numpy(), F.cpu().numpy()


@pytest.mark.parametrize("K", [160, 161, 1000, 4096])
@pytest.mark.parametrize("alpha,n", [(-1.5, 5), (0.25, 1), (0.25, 100), (1.0, 200), (1.0, 300),
                                     (1.5, 1000), (2.5, 2000), (6.0, 49)])
def test_forms_agree(ctx, orc, K, alpha, n):
    cells = [(alpha, n, 130, 11, 2, K), (1.2, 40, 70, 3, 0, K)]
    a, b = run(ctx, cells, "lane"), run(ctx, cells, "wave")
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    # sampled replicates against the oracle's fit of the same draws
    for rep in (0, 64, 129):
        x = torch.zeros(n, dtype=torch.int64, device="cuda")
        f = torch.zeros(n, dtype=torch.int32, device="cuda")
        ctx.sample_draws(alpha, n, 11, 2, rep, 1, x, f, kmax=K)
        torch.cuda.synchronize()
        r = orc.tz_fit(x.cpu().numpy(), K)
        assert abs(a[1][rep] - r["alpha_hat"]) <= 1e-10 * max(abs(r["alpha_hat"]), 1.0)
        assert abs(a[0][rep] - r["D"]) <= 1e-12
