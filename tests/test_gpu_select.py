"""GPU parity of the order statistics where their route changes: all values of
a cell gathered at once (2,048) or narrowed first, one workgroup per cell or
three launches (131,072), with and without ties, and more quantiles than one
pass takes.  Equal to the oracle's order statistic of the same D."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

QS = [(1, 1000), (1, 2), (9, 10), (95, 100), (99, 100), (999, 1000)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("R", [1, 64, 65, 2048, 2049, 8193, 131072, 131073])
@pytest.mark.parametrize("alpha,n,kmax", [(2.5, 200, 0), (3.5, 3, 0), (4.0, 10, 20), (1.3, 1, 0)])
def test_order_statistics(ctx, orc, R, alpha, n, kmax):
    cells = [(alpha, n, R, 7, 0, kmax), (alpha, n, max(1, R // 3), 8, 1, kmax)]
    d = torch.zeros(R + max(1, R // 3), dtype=torch.float64, device="cuda")
    q = np.asarray(ctx.simulate_cells(cells, quantiles=QS, d_out=d)).reshape(2, len(QS))
    D = d.cpu().numpy()
    for ci, Dc in enumerate((D[:R], D[R:])):
        for qi, (a, b) in enumerate(QS):
            assert q[ci, qi] == orc.quantile(Dc, a, b), (ci, a, b)
