"""The streaming selections' first thresholds (csrc/topn.hpp): rows too short to give enough keys, and rows of equal (masked) entries, of which
more lie above the first threshold than a buffer holds.  Checked as in test_gpu_selection_edges.py."""
import pytest
import torch

import test_gpu_selection_edges as edges

pytestmark = pytest.mark.gpu

SIZES = [(16, 200), (100, 256), (128, 193), (60, 57), (28, 29), (256, 256)]  # (s, top_k)
ROWS = [("random", 2000), ("masked", 2000), ("masked", 2048 * 4 + 8), ("late", 2048 * 9), ("constant", 2048 * 3), ("coarse", 2048 * 9)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("s,k", SIZES)
@pytest.mark.parametrize("order,V", ROWS)
def test_selections_from_their_start(dtype, s, k, order, V):
    edges.test_selections_at_their_edges(dtype, s, k, order, V)
