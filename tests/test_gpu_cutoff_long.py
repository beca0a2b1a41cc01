"""GPU parity of long replicates with a lower cutoff: 32-bit counts (n >=
65536), nearly all draws above the histogram, and replicate counts at which a
wave's share of the scratch holds just one replicate.  Every replicate's
outputs are written (they start as a mark), sampled ones match the oracle:
fingerprints and flags exact, alpha_hat 1e-10 relative, D 1e-12."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

XMIN = 10 ** 9
KEEP = 1 | 2 | 8  # ALL_ONES, TAIL_CAPPED, NOCONV
MARK = 0x5a5a5a5a


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,R", [(65535, 100), (65536, 100), (66533, 259), (123362, 103),
                                 (124359, 103)])
def test_every_replicate_is_written(ctx, orc, n, R):
    print("cutoff long", n, R, flush=True)
    D = torch.full((R,), float("nan"), dtype=torch.float64, device="cuda")
    A = torch.full_like(D, float("nan"))
    F = torch.full((R,), MARK, dtype=torch.int32, device="cuda")
    FP = torch.full((R,), MARK, dtype=torch.int64, device="cuda")
    q = ctx.simulate_cells([(2.5, n, R, 5, 1, 0, XMIN)], quantiles=[(9, 10)], d_out=D,
                           alpha_hat_out=A, flags_out=F, fingerprint_out=FP)
    d, a = D.cpu().numpy(), A.cpu().numpy()
    f, fp = F.cpu().numpy().view(np.uint32), FP.cpu().numpy().view(np.uint64)
    assert np.all(np.isfinite(d)) and np.all(np.isfinite(a)) and not np.any(f == MARK)
    assert q[0, 0] == orc.quantile(d, 9, 10)
    for rep in (0, 11, R - 1):
        r = orc.hz_simulate(2.5, XMIN, n, 5, 1, rep, 1)
        assert fp[rep] == r["fp"][0] and f[rep] & KEEP == r["flags"][0] & KEEP
        assert abs(a[rep] - r["alpha_hat"][0]) <= 1e-10 * r["alpha_hat"][0]
        assert abs(d[rep] - r["D"][0]) <= 1e-12
