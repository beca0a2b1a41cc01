"""What happens to a replicate with more large values than the scratch holds: one
that does not fit behind the others of its batch is drawn again first in the
next, one that does not fit at all is escalated, and one whose values fit but
not their copies takes the windows over all of them.  A call sizes its scratch
so that this takes twelve standard deviations, so the kernels are run here with
less (hostprobe/escalate.cpp); in the lane form escalation is ordinary.  Outputs
bit for bit those of the public call; the lanes' also against the wave form."""
import ctypes as C
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_6738_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def es(tmp_path_factory):
    from paper_1305_6738_amd import zpl
    zpl.lib()
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no C++ compiler"
    out = tmp_path_factory.mktemp("es") / "libes.so"
    subprocess.run([cxx, "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", str(HERE / "hostprobe" / "escalate.cpp"),
                    str(zpl.LIB_PATH), "-Wl,-rpath," + str(zpl.LIB_PATH.parent), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    vp = C.c_void_p
    L.es_run.argtypes = [C.c_double, C.c_int64, C.c_int32, C.c_uint64, C.c_uint32, C.c_uint32,
                         C.c_int64, C.c_uint32, C.c_int64, C.c_int32, vp, vp, vp, vp,
                         C.POINTER(C.c_uint32)]
    return L


def arrays(R):
    return (torch.full((R,), float("nan"), dtype=torch.float64, device="cuda"),
            torch.full((R,), float("nan"), dtype=torch.float64, device="cuda"),
            torch.full((R,), -1, dtype=torch.int32, device="cuda"),
            torch.zeros(R, dtype=torch.int64, device="cuda"))


def public(ctx, cell, form):
    D, A, F, FP = arrays(cell[2])
    ctx.simulate_cells([cell], quantiles=None, form=form, d_out=D, alpha_hat_out=A, flags_out=F,
                       fingerprint_out=FP)
    return [t.cpu().numpy() for t in (D, A, F, FP)]


# (alpha, n, R, K, xmin, room, words beyond one replicate's records and counts,
#  replicates escalated: none, some, all)
CASES = [(1.2, 600, 200, 0, 0, 8, 1500, "none"), (1.2, 600, 200, 0, 0, 8, 128, "some"),
         (1.2, 600, 60, 0, 0, 8, 16, "all"), (1.3, 65537, 30, 0, 0, 64, 6944, "some"),
         (-0.5, 400, 150, 4096, 0, 8, 2000, "none"), (-0.5, 400, 150, 4096, 0, 8, 352, "some"),
         (2.0, 300, 150, 0, 2000, 8, 1800, "none"), (2.0, 300, 150, 0, 2000, 8, 192, "some"),
         (1.3, 300, 60, 0, 5, 8, 64, "some"), (2.0, 300, 60, 0, 10 ** 6, 8, 64, "all"),
         # the copies do not fit: no place for the first level, or for its draws
         (2.0, 2000, 30, 0, 10 ** 6, 2000, 2010, "none"),
         (2.0, 2000, 30, 0, 10 ** 6, 2000, 2000 + 1600, "none"),
         (2.0, 2000, 30, 0, 10 ** 6, 2000, 2000 + 2600, "none"),
         (1.05, 2500, 30, 0, 0, 2500, 2510, "none"), (-0.5, 3000, 30, 4096, 0, 3000, 3010, "none")]


@pytest.mark.parametrize("case", CASES, ids=["a%g-n%d-K%d-x%d-w%d" % (c[0], c[1], c[3], c[4], c[6])
                                             for c in CASES])
def test_replicates_that_exceed_the_scratch(ctx, es, case):
    alpha, n, R, K, xmin, room, extra, escalated = case
    print("escalation", case, flush=True)
    want = public(ctx, (alpha, n, R, 21, 6, K, xmin), "heavy")
    got = arrays(R)
    out = (C.c_uint32 * 2)()
    torch.cuda.synchronize()
    assert es.es_run(alpha, n, R, 21, 6, K, xmin, room, extra, 48, *[t.data_ptr() for t in got],
                     out) == 0
    assert out[1] == 0
    assert {"none": out[0] == 0, "some": 0 < out[0] < R, "all": out[0] == R}[escalated], out[0]
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w)


@pytest.mark.parametrize("alpha,n,K", [(1.2, 1500, 0), (1.05, 300, 0), (0.25, 300, 4096),
                                       (0.25, 260, 1000), (-0.5, 400, 161), (0.25, 900, 100)])
def test_lanes_escalate(ctx, alpha, n, K):
    """About 224 and more values above a lane's column of 48: its slots are full
    in some replicates or in all."""
    R = 200
    for g, w in zip(public(ctx, (alpha, n, R, 3, 2, K), "lane"),
                    public(ctx, (alpha, n, R, 3, 2, K), "wave")):
        assert np.array_equal(g, w)
