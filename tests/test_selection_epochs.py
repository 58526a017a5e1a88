"""How long a selection goes without a barrier (csrc/selection_epochs.hpp).  The header is compiled for the host and its schedule is run,
with the buffers' sizes and the first thresholds of topn.hpp, on rows whose values rise along the vocabulary or have a band of early rounds
above the others: a buffer that runs full costs such a row a second, slow pass."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02620_amd", "csrc")
SOURCE = """
#include "selection_epochs.hpp"
using namespace difr;
extern "C" int epoch(int round, int first, int settled, int full) { return selection_epoch(round, first, settled, full); }
extern "C" int lik_first(int cap, int wide) { return likelihood_first_epoch(cap, wide); }
extern "C" int lik_settled(int cap, int wide) { return likelihood_settled(cap, wide); }
extern "C" int filt_first(int cap, int n, int primed, int wide) { return filtered_first_epoch(cap, n, primed != 0, wide); }
extern "C" int size(int which) { return which == 0 ? kTopCapSmall : which == 1 ? kTopCapMid : which == 2 ? kTopCapBig : which == 3 ? kLikEpoch : which == 4 ? kTopEpoch : kTopCapOne; }
"""
THREADS = 256
SMALL, MID, BIG, LIK, FILT, ONE = range(6)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("epochs")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    return C.CDLL(str(d / "s.so"))


def _rows(V, n, rise=0.0, band=0.0):
    """Scores of rows like a model's: -1.1 ln(rank), normal and Gumbel noise; rising by `rise` per 2048, or entries 2048 to 16,383 higher by `band`."""
    g = np.random.default_rng(V)
    for _ in range(n):
        x = -1.1 * np.log1p(g.permutation(V)) + g.standard_normal(V) - np.log(-np.log(g.random(V)))
        x += rise * (np.arange(V) // 2048)
        x[2048:16384] += band
        yield x


def _most(plan, v, n, wide, first, settled, full):
    """The most slots in use at the end of an epoch."""
    per = 2048 // wide
    rounds = v.size // per
    step = rounds // 4
    best = np.max([v[r * per:(r + 1) * per].reshape(THREADS, -1).max(1) for r in ([0, step, 2 * step, 3 * step] if step else [0])], axis=0)
    group = 4 if n <= 32 else (2 if n <= 100 else 1)
    theta = np.sort(best.reshape(-1, group).max(1))[-n]
    held, trigger, r, most = np.empty(0), max(n, 16), 0, 0
    while r < rounds:
        end = min(rounds, r + plan.epoch(r, first, settled, full))
        new = v[r * per:end * per]
        held = np.concatenate([held, new[new > theta]])
        most = max(most, held.size)
        if held.size >= trigger:
            held = np.sort(held)[-n:]
            theta, trigger = held[0], min(512, n + max(n, 16))
        r = end
    return most


def _likelihood(plan, v, n, wide):
    cap = plan.size(SMALL if n <= 64 else (MID if n <= 200 else BIG))
    return _most(plan, v, n, wide, plan.lik_first(cap, wide), plan.lik_settled(cap, wide), plan.size(LIK)) / cap


def _filtered(plan, v, n, wide):
    cap = plan.size(SMALL if n <= 64 else ONE)
    return _most(plan, v, n, wide, plan.filt_first(cap, n, 1, wide), plan.size(FILT), plan.size(FILT)) / cap


@pytest.mark.parametrize("wide", [1, 2])
@pytest.mark.parametrize("n", [16, 64, 128, 200, 256])
def test_ordinary_rows_have_room(plan, n, wide):
    # one row in thousands would make its launch wait for it: what some dozens of rows take at most stays well below the buffer
    for v in _rows(60 * 2048, 25):
        assert _likelihood(plan, v, n, wide) < 0.75
        assert _filtered(plan, v, n, wide) < 0.75


@pytest.mark.parametrize("wide", [1, 2])
@pytest.mark.parametrize("rounds,n,rise", [(8, 64, 0.5), (8, 50, 0.7), (8, 32, 1.0), (12, 32, 0.7), (12, 64, 0.7), (8, 128, 0.5), (12, 128, 0.5)])
def test_rising_rows(plan, rounds, n, rise, wide):
    for v in _rows(rounds * 2048, 10, rise=rise):
        assert _likelihood(plan, v, n, wide) <= 1


@pytest.mark.parametrize("wide", [1, 2])
@pytest.mark.parametrize("n", [16, 32, 50, 64, 100])
def test_band_of_early_rounds(plan, n, wide):
    for v in _rows(60 * 2048, 6, band=3.0):
        assert _likelihood(plan, v, n, wide) <= 1
        assert _filtered(plan, v, n, wide) <= 1


@pytest.mark.parametrize("wide", [1, 2])
@pytest.mark.parametrize("n", [65, 128, 200, 256])
def test_larger_filtered_selections(plan, n, wide):
    for row in (dict(rise=0.3), dict(band=3.0)):
        for v in _rows(8 * 2048, 6, **row):
            assert _filtered(plan, v, n, wide) <= 1


@pytest.mark.parametrize("n", [200, 256])
def test_second_round_of_a_band_and_what_waits(plan, n):
    # the filtered kernel: all of the first round's entries above the threshold may wait for the second round, all of which passes
    for v in _rows(16 * 2048, 150):
        best = np.max([v[r * 2048:(r + 1) * 2048].reshape(THREADS, -1).max(1) for r in (0, 4, 8, 12)], axis=0)
        assert np.count_nonzero(v[:2048] > np.sort(best)[-n]) + 2048 <= plan.size(ONE)


def test_schedule_is_plain(plan):
    for first, settled, full in ((1, 16, 16), (2, 8, 16), (4, 16, 16), (4, 8, 8), (6, 8, 8)):
        r, lens = 0, []
        while r < 64:
            lens.append(plan.epoch(r, first, settled, full))
            assert lens[-1] <= max(first, r) or r >= settled
            r += lens[-1]
        assert lens[0] == first and lens[-1] == full
