"""Shared rows whose parts do not all fit on the device at once (csrc/split.hip): the first parts keep their priority, the last share the issue
slots, and a row has the outputs it has in a batch whose parts do fit."""
import pytest
import torch

import paper_2511_02620_amd as difr

pytestmark = pytest.mark.gpu

# parts: 1050 of 3 or 4 rounds, 1200, 1282 (two to a row); four workgroups fit a compute unit with the rank, five without
SHAPES = [("bf16", 150, 50000, True), ("bf16", 300, 2048 * 31, True), ("bf16", 641, 2048 * 65, False), ("bf16", 641, 2048 * 65, True), ("f32", 641, 1024 * 130, True)]


@pytest.mark.parametrize("dtype,N,V,rank", SHAPES)
def test_rows_do_not_depend_on_what_fits(dtype, N, V, rank):
    g = torch.Generator(device="cuda").manual_seed(N)
    x = (3 * torch.randn(N, V, generator=g, device="cuda")).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    sid = torch.zeros(N, dtype=torch.int32, device="cuda")
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    seeds = torch.tensor([79], dtype=torch.int64, device="cuda")
    cg = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)
    ci = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)

    def score(a, b):
        at = (0.8, seeds, sid[a:b], pos[a:b])
        out = list(difr.score_both(x[a:b], *at, cg[a:b], ci[a:b], want_rank=rank))
        if not rank and V % 8 == 0:
            out += difr.score_both_admissible(x[a:b], *at, 1.5, cg[a:b], ci[a:b])
        return out

    whole, parts = score(0, N), [score(a, min(a + 40, N)) for a in range(0, N, 40)]
    for i, o in enumerate(whole):
        for k, w in o.items():
            if w is None:
                continue
            p = torch.cat([q[i][k] for q in parts])
            if k in ("margin", "argmax", "max_score", "claimed_score", "flags", "logit_rank", "u", "count", "log2_count"):
                assert torch.equal(w.view(torch.uint8), p.view(torch.uint8)), k
            else:  # sums over other parts: fp64 sums of the same fp32 terms, rounded to fp32
                assert torch.allclose(w, p, rtol=2e-6, atol=1e-7), k
