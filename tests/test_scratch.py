"""CPU check of the scratch that a simulation call's waves share
(zpl_scratch.hpp compiled for the host): whatever the number of replicates, the
room that the first replicate of a batch finds is at least what its cell asks
for.  A replicate that asks for all of its draws has no escalation launch
behind it, so one word too few would leave its outputs unwritten."""
import ctypes as C
import random
import shutil
import subprocess
from pathlib import Path

import pytest

HERE = Path(__file__).resolve().parent
N_CU = 256
BUDGET = 64 << 30


@pytest.fixture(scope="module")
def sc(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    assert cxx, "no C++ compiler"
    out = tmp_path_factory.mktemp("sc") / "libsc.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-fPIC", "-shared",
                    str(HERE / "hostprobe" / "scratch.cpp"), "-o", str(out)],
                   check=True, capture_output=True)
    L = C.CDLL(str(out))
    i64 = C.c_int64
    L.sc_area.restype = L.sc_first_room.restype = i64
    L.sc_area.argtypes = [i64, i64, i64, i64, C.c_uint64, C.c_int]
    L.sc_share.argtypes = [i64, i64, C.c_int, i64, C.c_int, C.POINTER(i64)]
    L.sc_first_room.argtypes = [i64, i64]
    return L


def share(sc, area, units, waves, room):
    out = (C.c_int64 * 2)()
    sc.sc_share(area, units, waves, room, N_CU, out)
    return out[0], out[1]


def first_room(sc, n, R, budget=BUDGET, waves=None):
    """Of one heavy-form cell whose room is all of its n draws."""
    waves = waves or sc.sc_waves_cut()
    area = sc.sc_area((R + 7) // 8, 0, n, 0, budget, N_CU)
    step = min(waves, max(1, (R + N_CU - 1) // N_CU))
    grid, stride = share(sc, area, (R + step - 1) // step, waves, n)
    assert 1 <= grid <= N_CU and grid * waves * stride <= area
    return sc.sc_first_room(stride, n)


@pytest.mark.parametrize("n,R", [(123362, 103), (124359, 103), (66533, 259), (72515, 521),
                                 (65535, 100), (65536, 100), (1 << 20, 7)])
def test_a_whole_replicate_fits(sc, n, R):
    assert first_room(sc, n, R) >= n


@pytest.mark.parametrize("budget", [1 << 28, 1 << 32, BUDGET])
def test_whole_replicates_fit_over_the_range(sc, budget):
    rng = random.Random(budget)
    for _ in range(20000):
        n = int(10 ** rng.uniform(0, 9.3))
        R = int(10 ** rng.uniform(0, 6))
        assert first_room(sc, n, R, budget) >= n, (n, R)
        # an escalated replicate, whatever the call holds besides
        area = sc.sc_area((R + 7) // 8, 0, n, 4096, budget, N_CU)
        grid, stride = share(sc, area, 64, sc.sc_esc_waves(), n)
        assert grid >= 1 and sc.sc_first_room(stride, n) >= n, (n, R)
