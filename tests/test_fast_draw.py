"""CPU check of the draw loops' 32-bit steps (zpl_math.hpp compiled for the
host): the guide bin by a uniform's first word is the bin by all 53 bits, the
threshold's words decide as the 53-bit comparison does, and the packed offsets
keep the bracket.  Integers: equal."""
import ctypes as C
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def fd(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(hipcc).exists():
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("fd") / "libfd.so"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(HERE / "hostprobe" / "fastdraw.cpp"), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    u64p = np.ctypeslib.ndpointer(np.uint64)
    L.fd_bins.restype = L.fd_thresholds.restype = C.c_int64
    L.fd_bins.argtypes = [u64p, C.c_int64, C.c_int, C.POINTER(C.c_int64)]
    L.fd_thresholds.argtypes = [u64p, u64p, C.c_int64]
    L.fd_offsets.restype = C.c_uint32
    L.fd_offsets.argtypes = [C.c_uint32]
    return L


def words(rng, octave):
    """Uniforms whose distance from 1 has its top bit at 31 - octave."""
    c = rng.integers(0, 2 ** 32, 4000, dtype=np.uint64) >> np.uint64(octave)
    c = np.concatenate([c, np.array([0, 1, 2, 2 ** 31 >> octave, (2 ** 32 >> octave) - 1], np.uint64)])
    hi = np.uint64(0xffffffff) - c
    lo = rng.integers(0, 2 ** 32, c.size, dtype=np.uint64)
    return np.concatenate([hi << np.uint64(32) | lo, hi << np.uint64(32),
                           hi << np.uint64(32) | np.uint64(0xffffffff)])


@pytest.mark.parametrize("octave", range(0, 32, 1))
def test_bins(fd, octave):
    rng = np.random.default_rng(octave)
    w = words(rng, octave)
    for sh in list(range(fd.fd_sh_max() + 1)) + [fd.fd_uniform()]:
        taken = C.c_int64(0)
        assert fd.fd_bins(w, w.size, sh, C.byref(taken)) == 0, sh
        if octave < 16:
            assert taken.value >= w.size // 2


@pytest.mark.parametrize("octave", [0, 1, 5, 20, 31])
def test_thresholds(fd, octave):
    rng = np.random.default_rng(100 + octave)
    w = words(rng, octave)
    m = w >> np.uint64(11) | np.uint64(1)
    for t in (m, m - np.uint64(1), m + np.uint64(1), m + np.uint64(2 ** 21), rng.permutation(m),
              np.full(m.size, 2 ** 53, np.uint64), np.zeros(m.size, np.uint64)):
        t = np.minimum(t, np.uint64(2 ** 53))
        assert fd.fd_thresholds(w, np.ascontiguousarray(t), w.size) == 0


def test_offsets(fd):
    for lo, hi in [(1, 1), (1, 2), (17, 18), (4096, 4096), (4096, 4097), (1, 4097)]:
        for mark in (0, 0x8000):
            o = fd.fd_offsets(lo | (mark | hi) << 16)
            assert (o & 0xffff) == 4 * (lo - 1)
            assert (o >> 16 & 0x7fff) == 4 * (hi - 1) and (o >> 31) == (1 if mark else 0)
