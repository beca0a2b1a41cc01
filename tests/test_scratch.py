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
    L.sc_area.restype = L.sc_first_room.restype = L.sc_need.restype = i64
    L.sc_need.argtypes = [i64]
    L.sc_parted.restype = i64
    L.sc_parted.argtypes = [i64, C.c_int, i64, C.c_uint64, C.c_int]
    L.sc_area.argtypes = [i64, i64, i64, i64, C.c_uint64, C.c_int]
    L.sc_share.argtypes = [i64, i64, C.c_int, i64, C.c_int, C.POINTER(i64)]
    L.sc_first_room.argtypes = [i64, i64]
    L.sc_place.argtypes = [i64, C.c_int, C.c_int, i64, i64, C.c_int, i64, i64, C.c_int,
                           C.POINTER(i64)]
    L.sc_split.argtypes = [i64, i64, C.c_int, i64, C.c_int, C.POINTER(i64)]
    return L


def share(sc, area, units, waves, room):
    out = (C.c_int64 * 3)()
    sc.sc_share(area, units, waves, room, N_CU, out)
    grid, stride, w = out
    assert 0 <= grid <= N_CU and 0 <= w <= waves and grid * w * stride <= area
    return grid, stride, w


def first_room(sc, n, R, budget=BUDGET, waves=None):
    """Of one heavy-form cell whose room is all of its n draws."""
    waves = waves or sc.sc_waves_cut()
    area = sc.sc_area((R + 7) // 8, 0, n, 0, budget, N_CU)
    step = min(waves, max(1, (R + N_CU - 1) // N_CU))
    grid, stride, w = share(sc, area, (R + step - 1) // step, step, n)
    assert grid >= 1 and w >= 1
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
        grid, stride, _ = share(sc, area, 64, sc.sc_esc_waves(), n)
        assert grid >= 1 and sc.sc_first_room(stride, n) >= n, (n, R)


@pytest.mark.parametrize("long_n", [10 ** 7, 3 * 10 ** 7, 10 ** 8])
def test_a_long_cell_leaves_the_device_to_the_others(sc, long_n):
    """24,000 replicates of 20,000 draws beside ten of long_n at alpha = 1.2 (a
    quarter of their draws above the histogram): the short ones keep a
    workgroup on every compute unit."""
    waves, units, room, long_room = sc.sc_waves(), 2000, 400, long_n // 4
    area = sc.sc_area(24000 // 8 + 2, 0, long_n, 4096, BUDGET, N_CU)
    grid, _, w = share(sc, area, units + 10, waves, long_room)
    assert grid * w < N_CU * waves // 2  # what one share for all would leave
    limit = C.c_int64()
    assert sc.sc_split(area, units + 10, waves, long_room, N_CU, C.byref(limit)) == 1
    assert sc.sc_need(room) <= limit.value < sc.sc_need(long_room)
    big, stride, _ = share(sc, area - area // 4, 10, waves, long_room)
    assert 1 <= big <= 10 and sc.sc_first_room(stride, long_n) >= long_room
    rest, stride, w = share(sc, area // 4, N_CU - big, waves, room)
    assert big + rest == N_CU and w == waves and sc.sc_first_room(stride, 20000) >= room


def test_equal_cells_are_not_split(sc):
    limit = C.c_int64()
    area = sc.sc_area(2500, 0, 10000, 4096, BUDGET, N_CU)
    assert sc.sc_split(area, 1700, sc.sc_waves(), 2200, N_CU, C.byref(limit)) == 0


def place(sc, total, lane_wgs, lane_waves, units, n_big, waves, max_room, small_room):
    stride = C.c_int64()
    r = sc.sc_place(total, lane_wgs, lane_waves, units, n_big, waves, max_room, small_room, N_CU,
                    C.byref(stride))
    return r, stride.value


@pytest.mark.parametrize("seed", range(4))
def test_places_do_not_overlap(sc, seed):
    """Lane units, long and short units of the other forms in every mixture."""
    rng = random.Random(seed)
    for _ in range(3000):
        n = int(10 ** rng.uniform(1, 8))
        lane_R = rng.choice([0, int(10 ** rng.uniform(0, 6))])
        block = rng.choice([64, 128, 192, 256, 384, 768])
        lane_wgs = min(N_CU, -(-lane_R // block))
        wave_R = rng.choice([0, int(10 ** rng.uniform(0, 6))])
        heavy_R = rng.choice([0, int(10 ** rng.uniform(0, 5))])
        sim_units = -(-lane_R // 768) + -(-wave_R // 768)
        if lane_wgs * block // 64 > max(1, min(sim_units, N_CU)) * 12:
            continue  # (the planner's lane units never outnumber what they bring in)
        total = sc.sc_area((heavy_R + 7) // 8, sim_units, n, 4096 if heavy_R else 0, BUDGET, N_CU)
        step = rng.randint(1, 12)
        units = -(-(wave_R + heavy_R) // step)
        n_big = rng.choice([0, 0, rng.randint(0, units)])
        room = rng.randint(1, n)
        small = room if n_big == 0 else min(room, rng.randint(1, 400))
        if n_big == units:
            small, n_big = room, 0
        r, _ = place(sc, total, lane_wgs, block // 64, units, n_big, step, room, small)
        if n_big == 0 and lane_wgs == 0:
            assert r == 0
        assert r in (0, 1), (seed, n, lane_wgs, block, units, n_big, step, room, small)


def test_both_kinds_share_a_place(sc):
    """A table of 12 exponents, 50,000 replicates of 100 draws each, ten in the
    lane form and two in the wave form: whole batches of 64 (384 words of records
    and 256 of counts a replicate)."""
    total = sc.sc_area(0, 792, 100, 0, BUDGET, N_CU)
    r, stride = place(sc, total, N_CU, 12, 1000, 0, sc.sc_waves(), 100, 100)
    assert r == 0 and stride >= 384 + 64 * 256 + 100


@pytest.mark.parametrize("n,room,R", [(1975, 1716, 3062), (1537, 1537, 2048), (2500, 2500, 3072),
                                      (2200, 2200, 10 ** 5), (7000, 7000, 3500), (65535, 65535, 1)])
def test_every_wave_of_a_unit_has_its_scratch(sc, n, room, R):
    """Replicates whose KS partitions its draws, in units of a replicate per wave:
    every wave holds one, so a unit takes one pass.  At most a sixteenth of the
    budget is brought in for it, and none for the shortest and longest rooms."""
    waves = sc.sc_waves_cut()
    step = min(waves, -(-R // N_CU))
    units = -(-R // step)
    more = sc.sc_parted(units, step, room, BUDGET, N_CU)
    area = max(sc.sc_area((R + 7) // 8, 0, n, 0, BUDGET, N_CU), more)
    grid, stride, w = share(sc, area, units, step, room)
    assert grid == min(units, N_CU) and w == step and stride >= sc.sc_need(room)
    assert 8 * more <= BUDGET // 16
    small = 1 << 28
    assert 8 * sc.sc_parted(units, step, room, small, N_CU) <= small // 16
    assert sc.sc_parted(units, step, 1536, BUDGET, N_CU) == 0
    assert sc.sc_parted(units, step, 65536, BUDGET, N_CU) == 0
