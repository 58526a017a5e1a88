"""The rules by which the host launches the row kernels (csrc/launch_rules.hpp), compiled for the host."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02620_amd", "csrc")
SOURCE = """
#include "launch_rules.hpp"
extern "C" int pace(int64_t groups, int resident, int64_t entries) { return difr::pace_from(groups, resident, entries); }
extern "C" int deep(int64_t N, int resident, int64_t rounds) { return difr::ipt_deep(N, resident, rounds); }
extern "C" int needed(int64_t N, int units) { return difr::pace_needed(N, units); }
extern "C" int f32_waves(int64_t N, int units, int rank, int64_t V) { return difr::gumbel_f32_waves(N, units, rank != 0, V); }
extern "C" unsigned idle(int64_t N, int units, int per_unit, int64_t rounds) { return difr::ipt_idle_lds(N, units, per_unit, rounds); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    lib = C.CDLL(str(d / "r.so"))
    lib.pace.argtypes = lib.deep.argtypes = [C.c_int64, C.c_int, C.c_int64]
    lib.needed.argtypes = [C.c_int64, C.c_int]
    lib.f32_waves.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int64]
    lib.idle.argtypes, lib.idle.restype = [C.c_int64, C.c_int, C.c_int, C.c_int64], C.c_uint
    return lib


@pytest.mark.parametrize("entries", [1, 5000, 32767, 32768, 151936])
def test_pace(rules, entries):
    for resident in (1024, 1280, 1536, 2048):
        for groups in (1, resident - 1, resident):               # all fit: all share
            assert rules.pace(groups, resident, entries) <= 0
        for groups in (resident + 1, resident + resident // 12):  # a few more than fit
            assert rules.pace(groups, resident, entries) == (groups if entries < 32768 else groups - resident)
        for groups in (resident + resident // 12 + 1, 3 * resident, 1 << 30):
            assert rules.pace(groups, resident, entries) == groups - resident
    assert rules.pace(1000, 0, entries) == 1000                   # not known: none is one of the last
    assert [rules.needed(N, 256) for N in (1, 256, 257, 16384)] == [0, 0, 1, 1]


def test_vectors_in_flight(rules):
    for N, rounds, deep in [(1, 5, 0), (1, 6, 1), (1024, 74, 1), (1025, 74, 0), (16384, 3, 0)]:
        assert rules.deep(N, 2048, rounds) == deep


@pytest.mark.parametrize("N", [1, 2048, 2049, 2304, 3000, 3072, 3500, 4096, 4500, 5000, 9000, 16384])
def test_workgroups_to_a_unit(rules, N):
    places = {p: -(-N // (256 * p)) * p for p in (8, 7, 6)}
    for rounds in (0, 4, 7, 8, 23, 24, 74):
        lds = rules.idle(N, 256, 8, rounds)
        if N <= 2048 or rounds < 8 or (rounds < 24 and N > 5120):
            assert lds == 0
            continue
        best = min(places, key=lambda p: (places[p], -p))
        assert lds == (0 if best == 8 else 163840 // best - 1024)
        assert lds == 0 or (163840 // (lds + 64) >= best and 163840 // (lds + 64) < best + 1)  # that many fit, and no more
    assert rules.idle(N, 256, 7, 74) == 0 and rules.idle(N, 0, 0, 74) == 0                       # not eight, or not known


def test_waves_of_the_fp32_stream(rules):
    for rank, fits in ((0, 1792), (1, 1536)):
        for N, waves in ((1, 1), (fits, 1), (fits + 1, 8), (2048, 8), (2049, 1), (5120, 1), (16384, 1)):
            assert rules.f32_waves(N, 256, rank, 128256) == waves
            assert rules.f32_waves(N, 256, rank, 1023) == 8
        assert rules.f32_waves(2048, 256, rank, 8191) == (1 if rank else 8)
        assert [rules.f32_waves(N, 256, rank, V) for N, V in ((5120, 30000), (5121, 30000), (5121, 65536))] == [1, 8, 1]
