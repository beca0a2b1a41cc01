"""The raw draws go through the steps of the simulation (first words, staged
tables, tail proposals one at a time), and its fingerprints and cap flags are
those of the draws in every form: for lengths that end a thread's four draws
anywhere, every layout of the guide, and tails that need double-double floors."""
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
    """Sum of splitmix64's finaliser over each row's values, mod 2^64."""
    z = x.astype(np.uint64)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return np.sum(z ^ (z >> np.uint64(31)), axis=1, dtype=np.uint64)


CELLS = [(2.5, 1, 0, 0), (2.5, 2, 0, 0), (2.5, 3, 0, 0), (1.5, 4, 0, 0), (1.5, 5, 0, 0),
         (1.01, 700, 0, 0), (1.2, 4001, 0, 0), (3.5, 1002, 0, 0), (0.25, 999, 1000, 0),
         (-2.0, 63, 4096, 0), (4.0, 130, 20, 0), (2.0, 1001, 0, 17), (1.3, 2003, 0, 10 ** 6),
         (2.5, 300, 0, 2)]


@pytest.mark.parametrize("alpha,n,K,xmin", CELLS)
def test_draws_are_the_simulation_s(ctx, alpha, n, K, xmin):
    count = 70
    x = torch.zeros(count * n, dtype=torch.int64, device="cuda")
    f = torch.zeros(count, dtype=torch.int32, device="cuda")
    ctx.sample_draws(alpha, n, 9, 4, 5, count, x, f, kmax=K, xmin=max(xmin, 1))
    torch.cuda.synchronize()
    v = x.cpu().numpy().reshape(count, n)
    assert v.min() >= max(xmin, 1) and (K == 0 or v.max() <= K)
    for form in (["heavy"] if xmin > 1 else ["lane", "wave", "heavy"]):
        fp = torch.zeros(count + 5, dtype=torch.int64, device="cuda")
        fl = torch.zeros(count + 5, dtype=torch.int32, device="cuda")
        ctx.simulate_cells([(alpha, n, count + 5, 9, 4, K, xmin)], quantiles=None, form=form,
                           fingerprint_out=fp, flags_out=fl)
        assert np.array_equal(fp.cpu().numpy().view(np.uint64)[5:], mix(v)), form
        assert np.array_equal(fl.cpu().numpy()[5:] & 2, f.cpu().numpy() & 2), form
