"""GPU parity of replicates with many draws above the 1,024 bins, which are
partitioned by bin in scratch (ks_many): around the count from which they are
(1,536), bins of 255 draws and more (a range of their own, down to single values
under the truncated law), ranges within ranges.  Against the oracle's fit of the
same draws, or for the longest the device's fit of them: alpha_hat 1e-10
relative, D 1e-12, fingerprints exact."""
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


def mix(x):
    """Sum of splitmix64's finaliser over the values, mod 2^64."""
    z = x.astype(np.uint64)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return np.sum(z ^ (z >> np.uint64(31)), dtype=np.uint64)


@pytest.mark.parametrize("alpha,n,R,K,xmin",
                         [(2.0, 1535, 40, 0, 10 ** 6), (2.0, 1537, 40, 0, 10 ** 6),
                          (2.0, 1600, 40, 0, 10 ** 6), (1.2, 12000, 70, 0, 0),
                          (3.0, 30000, 3, 0, 2 ** 40), (1.3, 20000, 9, 0, 100),
                          (60.0, 40000, 2, 0, 2 ** 21), (0.25, 20000, 9, 4096, 0),
                          (-0.5, 5000, 70, 4096, 0), (1.0, 70000, 2, 2000, 0),
                          (60.0, 16000000, 1, 0, 2 ** 21)])
def test_many_larger_draws(ctx, orc, alpha, n, R, K, xmin):
    print("many", alpha, n, K, xmin, flush=True)
    D = torch.full((R,), float("nan"), dtype=torch.float64, device="cuda")
    A = torch.full_like(D, float("nan"))
    FP = torch.zeros(R, dtype=torch.int64, device="cuda")
    ctx.simulate_cells([(alpha, n, R, 5, 3, K, xmin)], quantiles=None, form="heavy", d_out=D,
                       alpha_hat_out=A, fingerprint_out=FP)
    d, a, fp = D.cpu().numpy(), A.cpu().numpy(), FP.cpu().numpy().view(np.uint64)
    for rep in sorted({0, R // 2, R - 1}):
        x = torch.zeros(n, dtype=torch.int64, device="cuda")
        f = torch.zeros(1, dtype=torch.int32, device="cuda")
        ctx.sample_draws(alpha, n, 5, 3, rep, 1, x, f, kmax=K, xmin=max(xmin, 1))
        torch.cuda.synchronize()
        if n > 10 ** 6:
            r = ctx.fit(x, kmax=K, xmin=max(xmin, 1))
        else:
            xs = x.cpu().numpy()
            r = orc.tz_fit(xs, K) if K else (orc.hz_fit(xs, xmin) if xmin > 1 else orc.fit(xs))
            assert fp[rep] == mix(xs)
        assert abs(a[rep] - r["alpha_hat"]) <= 1e-10 * max(abs(r["alpha_hat"]), 1.0), rep
        assert abs(d[rep] - r["D"]) <= 1e-12, rep
