"""The search for the sampler's token from marks per wave: a mark every fourth round up to 128 rounds, fewer beyond, rows that end on
and beside a mark.  The rows and the comparison of test_gpu_ipt_search.py."""
import pytest
import torch

import test_gpu_ipt_search as base
from test_gpu_ipt_search import difr  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,rounds,extra", [
    (dt, r, e) for dt in (torch.bfloat16, torch.float32)
    for r, e in ((19, 5), (20, 0), (20, 3), (127, 2), (128, 0), (128, 9), (129, -1), (129, 1))])
def test_marks_per_wave(difr, dtype, rounds, extra):  # noqa: F811
    base.test_sampled_token_is_the_oracles(difr, dtype, rounds, extra)
