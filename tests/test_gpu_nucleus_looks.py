"""bf16 nuclei of rows about which the entries looked at beforehand say nothing, or something misleading: rows that are searched at once
because of them, with bins laid over a wrong span or from a reference far below, and rows that are counted and then searched after
all, for each of the reasons there are.  Which way a row goes is asserted with the look's rule in plain torch (nucleus_look.py); results
are compared with the oracle with the bounds of test_gpu_nucleus.py."""
import pytest
import torch

import nucleus_look
import test_gpu_nucleus as base

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


# kind: whether the rows are counted first (and then searched, unless "masked"), and the temperature
KINDS = {
    "masked": (True, 0.9),           # nothing usable is looked at: a pass of its own finds the reference
    "one value": (False, 0.9),       # a look of one value, no span for the bins
    "two values": (False, 0.9),      # a span of one step
    "far below, equal": (False, 0.9),  # the reference lies 120 below: the first pass starts again
    "far below": (True, 0.9),        # the same after counting
    "far above": (True, 0.9),        # outliers above a flat rest: counted
    "far above, equal": (False, 0.9),  # searched, with one bin that holds nearly all
    "spike": (True, 0.9),            # one entry of 130 and more that is not looked at
    "low": (True, 1.7),              # entries of -128 and below, not looked at, that carry mass
    "around zero": (True, 0.9),      # the cut among different values that share a counter
}


@pytest.mark.parametrize("V", [9000, 9003])
@pytest.mark.parametrize("kind", list(KINDS))
def test_looked_at_entries_unlike_the_row(difr, kind, V):
    N = 24
    counted, T = KINDS[kind]
    g = torch.Generator().manual_seed(len(kind) + V)
    seen = _seen(V)
    other = (~seen).nonzero().squeeze(1)
    x = torch.randn(N, V, generator=g) * 2.0
    noise = torch.randn(N, int(seen.sum()), generator=g)
    if kind == "masked":
        x[:, seen] = -float("inf")
    elif kind == "one value":
        x[:, seen] = 1.0
    elif kind == "two values":
        x[:, seen] = 1.0
        x[:, 7] = 1.0 + 2.0 ** -7
    elif kind == "far below, equal":
        x[:, seen] = -120.0
        x[:, 7] = -119.0
    elif kind == "far below":
        x[:, seen] = -110 + 3 * noise
    elif kind.startswith("far above"):
        x = x * 0.05 - 30.0
        x[:, seen] = 5.0 + (0.0 if "equal" in kind else 1.0) * noise
    elif kind == "spike":
        x[:, other[77]] = 130.0
        x[1::2, other[901]] = 131.0
    elif kind == "low":
        x = x * 8.0 - 95.0
        x[x < -127] = -127.0
        x[:, other[5:1500:3]] = -128.0 - 10 * torch.rand(N, len(other[5:1500:3]), generator=g)
    else:
        x = x.abs() * -1.0
        x[:, other[torch.randperm(len(other), generator=g)[:1500]]] = 2.0 ** -11 * torch.randn(N, 1500, generator=g)
    x = x.bfloat16()
    assert (nucleus_look.counted_first(x, V, T) == counted).all()
    logits = torch.full((N, -(-V // 8) * 8), float("nan"), dtype=torch.bfloat16, device=DEV)
    logits[:, :V] = x.to(DEV)
    row = torch.arange(N, dtype=torch.int32, device=DEV)
    claims = x.float().argmax(1).int()
    claims[1::2] = torch.randint(0, V, (N // 2,), generator=g, dtype=torch.int32)
    for p in (0.05, 0.3, 0.9, 0.99):
        print("nucleus looks", kind, V, p, flush=True)
        st, out = base._compare(difr, logits, V, T, torch.tensor([3], device=DEV), row * 0, row, claims.to(DEV), p)
        base.say("nucleus looks", kind, V, p, st)
        assert not (out["flags"] & 4).any()


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
