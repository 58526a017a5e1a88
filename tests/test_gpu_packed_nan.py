"""Rows that do not start on 16 bytes: every NaN is flagged on both sides, one with its sign bit set as much as one with it
clear, wherever it lies, and however the rows are scored (each estimator alone, the pair, the peaked pair; a workgroup per row,
and rows that are shared).  The flags and the argmax are those of the unfiltered kernel, which evaluates every entry."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [9, 2047, 20011, 49155, 99991])
def test_every_nan_of_a_packed_row_is_flagged(difr, dtype, V):
    N, S = 12, 2
    g = torch.Generator().manual_seed(V)
    x = (torch.randn(N, V, generator=g) * 2).to(dtype)
    bits = x.view(torch.int16 if dtype == torch.bfloat16 else torch.int32)
    clear, sign = (0x7FC0, -0x40) if dtype == torch.bfloat16 else (0x7FC00000, -0x400000)
    for row, (at, pattern) in enumerate([(0, sign), (V // 2, sign), (V - 1, sign), (V - 9, sign), (0, clear), (V // 2, clear),
                                         (V - 1, clear), (V - 9, sign + 1)]):
        bits[row, at] = pattern
    bad = torch.arange(N) < 8
    x[8, 1::2] = -float("inf")                    # (-inf and an ordinary row are not flagged)
    x[9] = -float("inf")
    x[9, V - 1] = 1.0
    assert torch.equal(x.isnan().any(1), bad)
    buf = torch.empty(N * V + 1, dtype=dtype, device=DEV)
    x = buf[1:].view(N, V).copy_(x)               # (V is odd: no row but by chance starts on 16 bytes)
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    at = (0.9, seeds, sid, pos)
    full = difr.gumbel_score(x, *at, unfiltered=True)
    claims = full["argmax"]
    full = difr.gumbel_score(x, *at, claims, unfiltered=True)
    print("packed NaN", dtype, V, flush=True)
    outs = {"gumbel": difr.gumbel_score(x, *at, claims), "gumbel, rank": difr.gumbel_score(x, *at, claims, want_rank=True),
            "ipt": difr.ipt_score(x, *at, claims)}
    for name, call in (("both", difr.score_both), ("peaked", difr.score_both_peaked)):
        for opt in ({}, dict(want_rank=True), dict(want_token=True)):
            outs["%s %s gumbel" % (name, opt)], outs["%s %s ipt" % (name, opt)] = call(x, *at, claims, claims, **opt)
    for name, o in outs.items():
        assert torch.equal((o["flags"] & 4).cpu() != 0, bad), (name, o["flags"])
        if "margin" in o:
            assert torch.equal(o["flags"], full["flags"]) and torch.equal(o["argmax"], full["argmax"]), name
