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
extern "C" int epoch(int round, int first, int full) { return selection_epoch(round, first, full); }
extern "C" int lik_first(int cap) { return likelihood_first_epoch(cap); }
extern "C" int filt_first(int cap, int n, int primed) { return filtered_first_epoch(cap, n, primed != 0); }
extern "C" int size(int which) { return which == 0 ? kTopCapSmall : which == 1 ? kTopCapMid : which == 2 ? kTopCapBig : which == 3 ? kLikEpoch : kTopEpoch; }
"""
PER, THREADS = 2048, 256  # entries of a round, bf16


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("epochs")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    return C.CDLL(str(d / "s.so"))


def _rows(rounds, n, rise=0.0, band=None, height=0.0):
    """Scores of rows like a model's: -1.1 ln(rank), normal and Gumbel noise."""
    g = np.random.default_rng(rounds)
    V = rounds * PER
    for _ in range(n):
        x = -1.1 * np.log1p(g.permutation(V)) + g.standard_normal(V) - np.log(-np.log(g.random(V)))
        x += rise * (np.arange(V) // PER)
        if band:
            x[band[0] * PER:band[1] * PER] += height
        yield x


def _runs_full(plan, v, n, cap, first, full):
    rounds = v.size // PER
    step = rounds // 4
    best = np.max([v[r * PER:(r + 1) * PER].reshape(THREADS, -1).max(1) for r in ([0, step, 2 * step, 3 * step] if step else [0])], axis=0)
    group = 4 if n <= 32 else (2 if n <= 100 else 1)
    theta = np.sort(best.reshape(-1, group).max(1))[-n]
    held, trigger, r = np.empty(0), max(n, 16), 0
    while r < rounds:
        end = min(rounds, r + plan.epoch(r, first, full))
        new = v[r * PER:end * PER]
        held = np.concatenate([held, new[new > theta]])
        if held.size > cap:
            return True
        if held.size >= trigger:
            held = np.sort(held)[-n:]
            theta, trigger = held[0], min(512, n + max(n, 16))
        r = end
    return False


@pytest.mark.parametrize("rounds,n,rise", [(8, 64, 0.5), (8, 50, 0.7), (8, 32, 1.0), (12, 32, 0.7), (12, 64, 0.7), (8, 128, 0.5), (12, 128, 0.5)])
def test_rising_rows(plan, rounds, n, rise):
    cap = plan.size(0 if n <= 64 else 1)
    full = [_runs_full(plan, v, n, cap, plan.lik_first(cap), plan.size(3)) for v in _rows(rounds, 10, rise=rise)]
    assert sum(full) == 0


@pytest.mark.parametrize("n", [16, 50, 100, 256])
def test_band_of_early_rounds(plan, n):
    lik, filt = plan.size(0 if n <= 64 else (1 if n <= 128 else 2)), plan.size(0 if n <= 64 else 2)
    for v in _rows(60, 6, band=(1, 8), height=3.0):
        assert not _runs_full(plan, v, n, lik, plan.lik_first(lik), plan.size(3))
        assert not _runs_full(plan, v, n, filt, plan.filt_first(filt, n, 1), plan.size(4))


def test_schedule_is_plain(plan):
    for first, full in ((1, 16), (2, 16), (4, 8)):
        r, lens = 0, []
        while r < 64:
            lens.append(plan.epoch(r, first, full))
            assert lens[-1] <= max(first, r) or r >= 8
            r += lens[-1]
        assert lens[-1] == full
