"""Calls of different forms in turn under one budget: each alone takes about
three quarters of it, and the context keeps what an earlier one allocated.  The
same replicates whatever came before, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def test_forms_in_turn_fit_the_budget():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    R = 256 * 768  # a workgroup's worth for every compute unit
    D = torch.zeros(R, dtype=torch.float64, device="cuda")
    got = []
    with Context(0, mem_budget_bytes=1 << 30) as ctx:
        for form in ("wave", "lane", "heavy", "lane", "wave"):
            D.zero_()
            ctx.simulate_cells([(2.5, 60, R, 1, 0)], quantiles=[(1, 2)], d_out=D, form=form)
            got.append(D.cpu().numpy())
            ctx.fit(np.arange(1, 60001))
    assert np.all(got[0] > 0)
    for g in got[1:]:
        assert np.array_equal(g, got[0])
