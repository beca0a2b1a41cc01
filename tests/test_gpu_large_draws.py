"""GPU parity of the batch form's larger draws (above its 1,024 bins) where
their route changes: none to 64 of them compared directly, windows of up to 255
grouped by bin, bins of 255 and more split; cutoffs at which half of the draws
are larger ones.  Sampled replicates against the oracle's fit of the same draws:
alpha_hat 1e-10 relative, D 1e-12."""
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


@pytest.mark.parametrize("alpha,n,xmin", [(1.8, 34, 798), (1.8, 130, 762), (1.8, 600, 762),
                                          (1.8, 3340, 762), (1.3, 3000, 5000), (3.0, 2000, 10 ** 6),
                                          (1.25, 3000, 1), (1.1, 20000, 1)])
def test_larger_draws(ctx, orc, alpha, n, xmin):
    R = 100
    D = torch.zeros(R, dtype=torch.float64, device="cuda")
    A = torch.zeros_like(D)
    ctx.simulate_cells([(alpha, n, R, 5, 3, 0, xmin)], quantiles=None, form="heavy", d_out=D,
                       alpha_hat_out=A)
    d, a = D.cpu().numpy(), A.cpu().numpy()
    for rep in (0, 1, 63, 99):
        x = torch.zeros(n, dtype=torch.int64, device="cuda")
        f = torch.zeros(n, dtype=torch.int32, device="cuda")
        ctx.sample_draws(alpha, n, 5, 3, rep, 1, x, f, xmin=xmin)
        torch.cuda.synchronize()
        xs = x.cpu().numpy()
        r = orc.hz_fit(xs, xmin) if xmin > 1 else orc.fit(xs)
        assert abs(a[rep] - r["alpha_hat"]) <= 1e-10 * r["alpha_hat"], rep
        assert abs(d[rep] - r["D"]) <= 1e-12, rep
