"""Host code of the library on a runtime of host memory (tests/native/
fake_hip.hpp): what it allocates and copies, and what it does when an
allocation fails.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1101_0876_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("host")

    def run(name, *args):
        exe = str(out / name)
        if not os.path.exists(exe):
            compile_program(name, exe)
        return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True, timeout=120).stdout.split()

    def compile_program(name, exe):
        subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "native", name + ".cpp"), os.path.join(PKG, "libpotts.so"),
                        f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined"], check=True)

    return run


def test_batch_after_a_failed_allocation(program):
    assert program("batch_alloc") == ["runs", "6", "misplaced", "0"]


# one launch: with a job on every CU (256), with the records of q = 200 to add up,
# or for a single sweep, whole lattices in LDS are faster than tiles
@pytest.mark.parametrize("count,L,q,n", [(512, 64, 9, 100), (512, 64, 200, 100), (256, 256, 9, 100), (128, 128, 200, 100),
                                         (1000, 16, 9, 100), (24, 64, 9, 1), (96, 64, 9, 100)])
def test_many_small_lattices_stay_in_lds(program, count, L, q, n):
    assert program("batch_routes", count, L, q, n) == ["1"]


@pytest.mark.parametrize("count,L,q,n", [(1, 256, 9, 100), (16, 256, 200, 100), (64, 192, 9, 100), (8, 128, 9, 100),
                                         (4, 512, 9, 100), (1, 2048, 9, 100)])
def test_few_lattices_take_tiles(program, count, L, q, n):
    assert 1 < int(program("batch_routes", count, L, q, n)[0]) < n


@pytest.mark.parametrize("count,L,q,n", [(64, 512, 9, 100), (48, 512, 200, 100), (300, 272, 9, 100), (1, 4096, 9, 100)])
def test_many_larger_lattices_share_strip_launches(program, count, L, q, n):
    assert 2 * n <= int(program("batch_routes", count, L, q, n)[0]) <= 2 * n + 4 + 2 * count


# tables of jobs and workgroups come on top: a few KiB
@pytest.mark.parametrize("jobs", [1, 2, 3, 4, 6])
def test_served_jobs_keep_to_the_budget(program, jobs):
    assert int(program("serve_budget", jobs)[0]) <= 64


def test_served_jobs_take_tiles_within_the_budget(program):
    strips, tiles = (int(program("serve_budget", jobs)[1]) for jobs in (4, 16))
    assert 0 < tiles < strips


def calls(program, *args):
    """(plain, cooperative) launches of each sweep call"""
    return [tuple(map(int, x.split("+"))) for x in program("choices", *args)]


# bands: one cooperative launch for up to 64 sweeps.  L = 4064, whose rows are no
# whole waves of items, is faster on tiles; at L = 2048 they are from 16 sweeps on,
# 32 on a new state
def test_band_choice(program):
    assert [c for _, c in calls(program, "square", 4096, 6, 1, 64, 65)] == [1, 1, 2]
    assert [c for _, c in calls(program, "square", 4064, 6, 1, 64)] == [0, 0]
    assert [c for _, c in calls(program, "square", 1984, 6, 64)] == [0]
    assert [c for _, c in calls(program, "square", 2048, 200, 31, 32, 15, 16)] == [0, 1, 0, 1]


# Launches of a call: colour-split 2 a sweep, a cleared record and a fold, and 1 to
# pack the rows; tiles one for up to eight sweeps and a fold, and 1 to unpack the
# planes.  Calls of one sweep and longer ones do not move the lattice back and
# forth, and L = 4640 takes the planes only.
def test_short_calls_stay_where_the_lattice_is(program):
    assert [n for n, _ in calls(program, "square", 4512, 6, 1, 2, 3, 7, 1)] == [5, 6, 8, 16, 4]
    assert [n for n, _ in calls(program, "heat bath", 3968, 6, 1, 4, 11)] == [5, 10, 24]
    assert calls(program, "heat bath", 3968, 6, 1, 16)[1][0] < 16
    assert calls(program, "heat bath", 3968, 6, 4)[0][0] < 10
    assert calls(program, "square", 4512, 6, 3)[0][0] < 6
    assert calls(program, "square", 4128, 6, 2)[0][0] < 6
    assert calls(program, "square", 4128, 6, 1, 4)[1][0] < 8
    assert calls(program, "square", 4640, 6, 16)[0][0] == 35


def test_one_sweep_of_a_small_lattice(program):
    assert [n for n, _ in calls(program, "square", 112, 6, 1, 2)] == [1, 2]  # LDS-resident; a tile launch and its fold


# cubes: the chunk kernel has 2 launches a sweep and one to clear the record, the
# colour-split kernel a fold, a pack and an unpack besides the 2 a sweep
def test_small_cubes(program):
    for L, want in ((68, [3, 5, 101]), (72, [3, 7, 102]), (76, [3, 7, 102]), (80, [5, 6, 102])):
        assert [n for n, _ in calls(program, "cube", L, 200, 1, 2, 50)] == want, L


# the host copy of the last record: not for a lattice that is looked at a few
# times, and never where the kernel does not fill it
@pytest.mark.parametrize("L,want", [(64, "000111"), (112, "000111"), (1000, "000111"), (4864, "000000")])
def test_pinned_record_after_some_observations(program, L, want):
    assert "".join(program("observations", L)) == want


# L % 32 != 0: the planes hold a lattice of the library's own between calls; in the
# caller's buffers every call packs and unpacks, or stays in the strip kernel (a
# cleared record, 2 a sweep and a fold) where it is too short to make up for it
def test_ragged_planes(program):
    assert [n for n, _ in calls(program, "square", 5008, 6, 1, 1, 2)] == [5, 4, 6]
    assert [n for n, _ in calls(program, "square", 8016, 6, 1, 1)] == [5, 4]
    assert [n for n, _ in calls(program, "buffers", 5008, 6, 1, 2)] == [4, 8]
    assert [n for n, _ in calls(program, "buffers", 7184, 6, 3, 4)] == [8, 12]
    assert [n for n, _ in calls(program, "buffers", 8016, 6, 23, 24)] == [48, 52]
    assert [n for n, _ in calls(program, "buffers", 5012, 6, 1)] == [6]  # one 4-byte chunk a lane otherwise


# a kernel that needs no memory takes the lattice where there is none (L = 64's
# drawn words, the bands and the planes of L^2 bytes apart)
@pytest.mark.parametrize("kind,L,q,n", [("square", 80, 6, 10), ("square", 96, 200, 3), ("square", 112, 9, 5),
                                        ("square", 100, 6, 9), ("square", 256, 40, 9), ("square", 1000, 6, 9),
                                        ("square", 1024, 6, 9), ("square", 5008, 6, 2), ("square", 4740, 6, 2),
                                        ("heat bath", 100, 6, 9), ("heat bath", 1000, 40, 2), ("heat bath", 4740, 6, 1),
                                        ("cube", 100, 3, 4), ("cube", 60, 3, 4), ("nnn", 504, 9, 9), ("nnn", 4092, 200, 2)])
def test_sweeps_without_memory(program, kind, L, q, n):
    assert program("sweep_alloc", kind, L, q, n)[0] == "14/14"


def test_served_job_without_memory_for_tiles(program):
    assert program("serve_alloc") == ["0"] * 4
