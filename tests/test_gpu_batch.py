"""GPU parity of the batched heavy form (zpl_batch.hpp): the KS distance by
bounds against the oracle's walk over every distinct value, at the sizes where
the batch can go wrong -- one draw, the 64-draw and 16-bit/32-bit count edges,
replicates whose larger draws fill several windows of the gather, cutoffs on
both sides of the head sums (16) and of the relative survival values (17).

Bar: fingerprints and flags exact, alpha_hat within 1e-10, D within 1e-12 (the
rounding of both sides' sums at D <= 1), as for the other forms.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KEEP_FLAGS = 1 | 2 | 8  # ALL_ONES, TAIL_CAPPED, NOCONV


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


def run(ctx, cells, form):
    R = sum(c[2] for c in cells)
    d, a = (torch.zeros(R, dtype=torch.float64, device="cuda") for _ in range(2))
    f = torch.zeros(R, dtype=torch.int32, device="cuda")
    fp = torch.zeros(R, dtype=torch.int64, device="cuda")
    ctx.simulate_cells(cells, quantiles=None, d_out=d, alpha_hat_out=a, flags_out=f,
                       fingerprint_out=fp, form=form)
    torch.cuda.synchronize()
    return {"D": d.cpu().numpy(), "alpha_hat": a.cpu().numpy(),
            "flags": f.cpu().numpy().view(np.uint32), "fp": fp.cpu().numpy().view(np.uint64)}


# (alpha, n, replicates, xmin)
CELLS = [(2.5, 1, 200, 0), (1.5, 2, 200, 0), (1.2, 63, 150, 0), (1.2, 129, 150, 0),
         (1.02, 700, 60, 0), (3.5, 1000, 130, 0), (1.5, 4097, 40, 0), (1.3, 20000, 12, 0),
         (1.25, 60000, 5, 0), (1.6, 65535, 5, 0), (1.6, 65536, 5, 0), (2.2, 300001, 3, 0),
         (2.0, 500, 60, 2), (2.5, 500, 60, 15), (2.5, 500, 60, 16), (2.5, 500, 60, 17),
         (2.5, 500, 60, 18), (1.4, 3000, 20, 100), (2.2, 2000, 20, 50000),
         (6.0, 300, 60, 12)]


@pytest.mark.parametrize("cell", CELLS, ids=["a%g-n%d-x%d" % (c[0], c[1], c[3]) for c in CELLS])
def test_batched_replicates_match_the_oracle(ctx, orc, cell):
    alpha, n, R, xmin = cell
    print("batch", cell, flush=True)
    sys.stdout.flush()
    g = run(ctx, [(alpha, n, R, 77, 5, 0, xmin)], "heavy")
    ref = (orc.hz_simulate(alpha, xmin, n, 77, 5, 0, R) if xmin > 1
           else orc.simulate(alpha, n, 77, 5, 0, R))
    assert np.array_equal(g["fp"], ref["fp"])
    keep = KEEP_FLAGS if xmin > 1 else 3
    assert np.array_equal(g["flags"] & keep, ref["flags"] & keep)
    assert np.max(np.abs(g["alpha_hat"] - ref["alpha_hat"]) / ref["alpha_hat"]) < 1e-10
    assert np.max(np.abs(g["D"] - ref["D"])) < 1e-12
