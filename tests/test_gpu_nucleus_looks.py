"""bf16 nuclei of rows about which the entries looked at beforehand say nothing, or something misleading: rows that are searched at once
because of them, with bins laid over a wrong span or from a reference far below, and rows that are counted and then searched after
all, for each of the reasons there are.  Which way a row goes is asserted with the look's rule in plain torch (nucleus_look.py); results
are compared with the oracle with the bounds of test_gpu_nucleus.py."""
import pytest
import torch

import nucleus_look

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _seen(V):
    """Mask of the positions looked at."""
    seen = torch.zeros(-(-V // 8) * 8, dtype=torch.bool)
    seen.view(-1, 8)[nucleus_look.looked_at(V)] = True
    return seen[:V]


@pytest.mark.parametrize("V", [2048, 9003])
def test_undefined_rows_that_are_counted_first(difr, V):
    """A NaN of either sign, and +inf, at a place that is not looked at (or the row's only ones looked at: 2048 entries are all seen)."""
    bits = [0x7FC0, -1, 0x7F80, 0x7F81, -127]
    x = torch.randn(len(bits), -(-V // 8) * 8, generator=torch.Generator().manual_seed(V)).bfloat16()
    at = int((~_seen(V)).nonzero()[9]) if V > 2048 else 77
    for r, b in enumerate(bits):
        x.view(torch.int16)[r, at] = b
    row = torch.arange(len(bits), dtype=torch.int32, device=DEV)
    print("nucleus looks, undefined", V, flush=True)
    out = difr.ipt_score_filtered(x.to(DEV)[:, :V], 0.8, torch.tensor([5], device=DEV), row * 0, row, row * 0, top_k=0, top_p=0.9, V=V,
                                  want_token=True)
    assert (out["flags"] == 4).all() and (out["kept"] == 0).all() and out["dist"].isnan().all() and (out["ipt_token"] == -1).all()
