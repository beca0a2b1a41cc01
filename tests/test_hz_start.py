"""CPU checks of what the cutoff law's MLE takes for granted away from its edge
(zpl_math.hpp compiled for the host): mu(64) - ln xmin stays below 1/32, so a
larger mean has its root in the bracket; there the solver ends at the oracle's
root (its own stopping rule, 2^-40) within the conditioning of eq. 2 and in
few steps; and the truncated law's solver from its start does too."""
import ctypes as C
import math
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def hm(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(hipcc).exists():
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("hz") / "libhz.so"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(HERE / "hostprobe" / "hostmath.cpp"), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    L.hm_hurwitz3.argtypes = [C.c_double, C.c_int64, C.POINTER(C.c_double)]
    L.hm_mle_hz_it.restype = C.c_double
    L.hm_mle_hz_it.argtypes = [C.c_double, C.c_int64, C.POINTER(C.c_uint32), C.POINTER(C.c_int)]
    L.hm_mle_trunc_it.restype = C.c_double
    L.hm_mle_trunc_it.argtypes = [C.c_double, C.c_uint32, C.POINTER(C.c_uint32),
                                  C.POINTER(C.c_int)]
    return L


def stats(hm, s, xmin):
    out = (C.c_double * 3)()
    hm.hm_hurwitz3(s, xmin, out)
    r = out[1] / out[0]
    return -r, out[2] / out[0] - r * r  # mean and variance of ln X


def test_the_edge_is_below(hm):
    for xmin in list(range(2, 400)) + [10 ** k for k in range(3, 13)] + [2 ** 40]:
        assert stats(hm, 64.0, xmin)[0] - math.log(xmin) < 1 / 32, xmin


@pytest.mark.parametrize("xmin", [2, 3, 9, 16, 17, 18, 100, 5000, 10 ** 9, 2 ** 40])
def test_cutoff_roots(hm, orc, xmin):
    rng = np.random.default_rng(xmin % 1000)
    for t in np.concatenate([[0.03126, 0.0313], 10 ** rng.uniform(math.log10(0.0313), 1.3, 400)]):
        m = math.log(xmin) + float(t)
        f, it = C.c_uint32(0), C.c_int(0)
        a = hm.hm_mle_hz_it(m, xmin, C.byref(f), C.byref(it))
        ao, fo = orc.hz_mle(m, xmin)
        assert f.value & 8 == fo & 8 == 0
        assert it.value <= 20
        # both sides fix the root to the rounding of m and mu: 32 of them
        tol = 32 * 2.0 ** -53 * m / stats(hm, ao, xmin)[1] + 2.0 ** -50 * ao
        assert abs(a - ao) <= tol, (t, a, ao)


@pytest.mark.parametrize("K", [2, 5, 20, 160, 161, 1000, 4096])
def test_truncated_roots(hm, orc, K):
    rng = np.random.default_rng(K)
    for x in rng.uniform(0.02, 0.98, 300):
        m = float(x) * math.log(K)
        f, it = C.c_uint32(0), C.c_int(0)
        a = hm.hm_mle_trunc_it(m, K, C.byref(f), C.byref(it))
        ao, fo = orc.tz_mle(m, K)
        assert f.value & 8 == fo & 8
        assert it.value <= 12
        assert abs(a - ao) <= 1e-10 * max(abs(ao), 1.0), (x, a, ao)
