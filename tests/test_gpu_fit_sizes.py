"""GPU parity of the dataset fits where their route changes: one workgroup or
many (32,768 values), the values counted by value (up to 4,096) and those
sorted, one sorted run or passes of merges (4,096 and 65,536 larger values),
few candidates with shared distances or many (128).  Against the oracle with
its stated tolerances: alpha_hat 1e-10 relative, D 1e-12, flags and n_tail
equal."""
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


def close(r, ref, case):
    assert abs(r["alpha_hat"] - ref["alpha_hat"]) <= 1e-10 * max(abs(ref["alpha_hat"]), 1.0), case
    assert abs(r["D"] - ref["D"]) <= 1e-12, case
    assert r["flags"] & FLAGS == ref["flags"] & FLAGS, case


def data(kind, n):
    rng = np.random.default_rng(n)
    if kind == "law":
        return np.minimum(rng.zipf(1.7, n), 2 ** 62).astype(np.int64)
    if kind == "large":  # every value sorted, with many copies
        return (4095 + rng.integers(1, 3000, n)).astype(np.int64)
    if kind == "one":    # every value the same, sorted
        return np.full(n, 5000, np.int64)
    if kind == "huge":   # spread over the whole type, its largest value included
        x = np.floor(np.exp(rng.uniform(0, 43.6, n))).astype(np.int64)
        x[:3] = 2 ** 63 - 1
        return x
    raise AssertionError(kind)


@pytest.mark.parametrize("n", [1, 2, 513, 4097, 32767, 32768, 32769, 65537, 140000])
@pytest.mark.parametrize("kind", ["law", "large", "one", "huge"])
def test_fit_sizes(ctx, orc, kind, n):
    x = data(kind, n)
    close(ctx.fit(x), orc.fit(x), (kind, n))
    d = ctx.fit(torch.from_numpy(x).cuda())
    close(d, orc.fit(x), (kind, n, "device"))
    if n > 40000:  # a value out of range is found wherever it is
        x[n - 1] = 0
        from paper_1305_6738_amd import ZplError
        with pytest.raises(ZplError):
            ctx.fit(x)


@pytest.mark.parametrize("n", [300, 32767, 40000])
@pytest.mark.parametrize("K", [2, 17, 160, 161, 4096])
def test_fit_truncated_sizes(ctx, orc, K, n):
    rng = np.random.default_rng(K)
    x = (rng.zipf(1.2, n) % K + 1).astype(np.int64)
    close(ctx.fit(x, kmax=K), orc.tz_fit(x, K), (K, n))


@pytest.mark.parametrize("n", [300, 32767, 70000])
@pytest.mark.parametrize("count", [1, 128, 129])
def test_scan_sizes(ctx, orc, n, count):
    x = data("law", n)
    edges = [1, 2, 16, 17, 18, 4095, 4096, 4097, 4098, 5000, 10 ** 7, 2 ** 40]
    cand = np.array([4097] if count == 1 else edges + list(range(20, 20 + count - len(edges))))
    g, r = ctx.fit_scan(x, cand), orc.hz_scan(x, cand)
    assert np.array_equal(g["n_tail"], r["n_tail"])
    fin = np.isfinite(r["D"])
    assert np.array_equal(np.isfinite(g["D"]), fin)
    assert np.all(np.abs(g["D"][fin] - r["D"][fin]) <= 1e-12)
    assert np.all(np.abs(g["alpha_hat"][fin] - r["alpha_hat"][fin]) <= 1e-10 * r["alpha_hat"][fin])
    assert np.array_equal(g["flags"] & FLAGS, r["flags"] & FLAGS)
