"""CPU check of the truncated law's survival sums by Euler-Maclaurin
(zpl_math.hpp compiled for the host) against sums in extended precision, at the
smallest K the form takes for each exponent and up to the table's end.
Tolerance: a power's argument |s| ln k is rounded once (relative error
|s| ln K 2^-53 of the power, for the sum and for the normaliser), plus 64
roundings each."""
import ctypes as C
import math
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def tt(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(hipcc).exists():
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("tt") / "libtt.so"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(HERE / "hostprobe" / "trunctail.cpp"), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    L.tt_em.argtypes = [C.c_double, C.c_uint32]
    L.tt_sums.argtypes = [C.c_double, C.c_uint32, C.POINTER(C.c_double)]
    return L


@pytest.mark.parametrize("s", [-64.0, -20.0, -5.0, -3.3, -1.0, 0.0, 1e-9, 0.5, 1 - 1e-12, 1.0,
                               1 + 1e-12, 1.1, 2.0, 4.375, 8.0, 30.0, 64.0])
def test_survival_sums(tt, s):
    first = next(K for K in range(17, 4097) if tt.tt_em(s, K))
    for K in sorted({first, first + 1, 161, 500, 1000, 4096}):
        if K < first:
            continue
        out = (C.c_double * (K + 1))()
        tt.tt_sums(s, K, out)
        k = np.arange(1, K + 1, dtype=np.longdouble)
        top = np.log(np.longdouble(K)) if s < 0 else np.longdouble(0)
        w = np.exp(-np.longdouble(s) * (np.log(k) - top))
        suf = np.concatenate([np.cumsum(w[::-1])[::-1], [0]])
        o = np.array(out).astype(np.longdouble)
        tol = 2 * (abs(s) * math.log(K) + 64) * 2.0 ** -53
        assert np.abs(o / o[0] - suf / suf[0]).max() <= tol, K
