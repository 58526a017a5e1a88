"""The rules by which the host launches the row kernels (csrc/launch_rules.hpp), compiled for the host."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02620_amd", "csrc")
SOURCE = """
#include "launch_rules.hpp"
extern "C" int pace(int64_t groups, int resident, int64_t entries) { return difr::pace_from(groups, resident, entries); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    lib = C.CDLL(str(d / "r.so"))
    lib.pace.argtypes = [C.c_int64, C.c_int, C.c_int64]
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
