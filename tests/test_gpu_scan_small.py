"""GPU parity of scans of small datasets, which each candidate's workgroup
counts and sorts itself (up to 1,024 values and 512 candidates): at those edges,
with every value among the sorted ones, with the type's largest value, with
cutoffs at the lines of the survival sums and above every value, and with values
out of range.  Oracle's tolerances: alpha_hat 1e-10 relative, D 1e-12, flags and
n_tail equal."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

FLAGS = 1 | 8  # ALL_ONES, NOCONV


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


def data(kind, n):
    rng = np.random.default_rng(n)
    if kind == "law":
        return np.minimum(rng.zipf(1.5, n), 2 ** 62).astype(np.int64)
    if kind == "large":
        return (4095 + rng.integers(1, 300, n)).astype(np.int64)
    x = np.floor(np.exp(rng.uniform(0, 43.6, n))).astype(np.int64)
    x[:2] = 2 ** 63 - 1
    return x


@pytest.mark.parametrize("n", [1, 2, 63, 1023, 1024, 1025])
@pytest.mark.parametrize("count", [1, 512, 513])
@pytest.mark.parametrize("kind", ["law", "large", "huge"])
def test_small_scans(ctx, orc, kind, n, count):
    x = data(kind, n)
    edges = [1, 2, 16, 17, 18, 4095, 4096, 4097, 4098, 4200, 10 ** 7, 2 ** 40]
    cand = np.array([1] if count == 1 else (edges + list(range(20, 20 + count)))[:count])
    g, r = ctx.fit_scan(x, cand), orc.hz_scan(x, cand)
    assert np.array_equal(g["n_tail"], r["n_tail"])
    fin = np.isfinite(r["D"])
    assert np.array_equal(np.isfinite(g["D"]), fin)
    assert np.all(np.abs(g["D"][fin] - r["D"][fin]) <= 1e-12)
    assert np.all(np.abs(g["alpha_hat"][fin] - r["alpha_hat"][fin]) <= 1e-10 * r["alpha_hat"][fin])
    assert np.array_equal(g["flags"] & FLAGS, r["flags"] & FLAGS)


@pytest.mark.parametrize("n", [1, 700, 1024])
def test_small_scan_refusals(ctx, n):
    from paper_1305_6738_amd import ZplError
    x = data("law", n)
    with pytest.raises(ZplError):  # no value at or above the cutoff
        ctx.fit(np.minimum(x, 50), xmin=51)
    x[n - 1] = 0
    with pytest.raises(ZplError):
        ctx.fit_scan(x, [1, 2, 3])
