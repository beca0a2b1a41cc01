"""CPU check of the MLE's tabulated start (zpl_math.hpp compiled for the host):
over every mean of logarithms a sample can have, and at the ends of the table,
one evaluation of the zeta sums ends at the root that the general iteration
finds.  Tolerance: both roots carry the rounding of mu, a few 2^-53 of alpha
(4 ulps allowed); outside the table more evaluations end there too."""
import ctypes as C
import math
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def ms(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(hipcc).exists():
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("ms") / "libms.so"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(HERE / "hostprobe" / "mlestart.cpp"), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    L.ms_general.restype = L.ms_start.restype = C.c_double
    L.ms_general.argtypes = [C.c_double, C.POINTER(C.c_uint32)]
    L.ms_start.argtypes = [C.c_double, C.POINTER(C.c_uint32), C.POINTER(C.c_int)]
    return L


@pytest.mark.parametrize("lo,hi,count", [(math.log(2) / 2 ** 31, 1e-6, 2000), (1e-6, 0.1, 4000),
                                         (0.1, 3.0, 6000), (3.0, 63 * math.log(2), 4000),
                                         (1e-12, 1e-10, 50), (46.0, 60.0, 50)])
def test_tabulated_start_gives_the_general_root(ms, lo, hi, count):
    rng = np.random.default_rng(5)
    m = np.exp(rng.uniform(math.log(lo), math.log(hi), count))
    inside = lo >= math.log(2) / 2 ** 31 and hi <= 44.0
    fl, fg, it = C.c_uint32(0), C.c_uint32(0), C.c_int(0)
    for v in np.concatenate([[lo, hi], m]):
        fl.value = fg.value = 0
        a, b = ms.ms_start(v, C.byref(fl), C.byref(it)), ms.ms_general(v, C.byref(fg))
        assert fl.value == fg.value
        assert abs(a - b) <= 4 * 2.0 ** -53 * b
        if inside:
            assert it.value == 1
