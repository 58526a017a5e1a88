"""Rows take a priority from their place in the grid and from how much of them is left (csrc/difr_device.hpp, RowPace): batches that
end below, at and above the number of rows the device holds at once give every row the outputs it has in a batch of another size."""
import pytest
import torch

import paper_2511_02620_amd as difr

pytestmark = pytest.mark.gpu

# rounds of 2048 (bf16) or 1024 (fp32) entries: fewer than three, a third that is no whole number, ragged ends
SHAPES = [("bf16", 1281, 2048 * 2 + 8), ("bf16", 1025, 2048 * 7 + 520), ("bf16", 2561, 2048 * 16), ("bf16", 1300, 2048 * 5 + 3),
          ("f32", 1537, 1024 * 4 + 4), ("f32", 1793, 1024 * 17)]


@pytest.mark.parametrize("dtype,N,V", SHAPES)
def test_rows_do_not_depend_on_their_batch(dtype, N, V):
    g = torch.Generator(device="cuda").manual_seed(N + V)
    x = (3 * torch.randn(N, V, generator=g, device="cuda")).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    sid = torch.zeros(N, dtype=torch.int32, device="cuda")
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    seeds = torch.tensor([77], dtype=torch.int64, device="cuda")
    cg = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)
    ci = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)

    def score(a, b):
        at = (0.8, seeds, sid[a:b], pos[a:b])
        out = [difr.gumbel_score(x[a:b], *at, cg[a:b], want_rank=True)]
        out += difr.score_both(x[a:b], *at, cg[a:b], ci[a:b], want_token=True)
        out += difr.score_both(x[a:b], *at, cg[a:b], ci[a:b], want_rank=True)
        if V % 8 == 0:
            out += difr.score_both_admissible(x[a:b], *at, 1.5, cg[a:b], ci[a:b])
        return [(k, v) for o in out for k, v in o.items() if v is not None]

    whole = score(0, N)
    cut = N // 3
    for (k, w), (_, p), (_, q) in zip(whole, score(0, cut), score(cut, N)):
        both = torch.cat([p, q])
        assert torch.equal(w.view(torch.uint8), both.view(torch.uint8)), k
