"""Token-IPT-DiFR alone keeps one or three vectors in flight and lets eight, seven or six workgroups share a compute unit, depending on
the number of rows (csrc/ipt.hip): a row has the same outputs in every batch, and they are those of the one-pass kernel."""
import pytest
import torch

import paper_2511_02620_amd as difr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rounds,extra", [(0, 900), (1, 0), (2, 8), (3, 1), (4, 0), (5, 2040), (16, 0), (17, 3)])
def test_rows_do_not_depend_on_their_batch(dtype, rounds, extra):
    per_round = 2048 if dtype == "bf16" else 1024
    N, V = 2100, rounds * per_round + min(extra, per_round - 1)
    g = torch.Generator(device="cuda").manual_seed(rounds)
    x = (2 * torch.randn(N, V, generator=g, device="cuda")).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    sid = torch.zeros(N, dtype=torch.int32, device="cuda")
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    seeds = torch.tensor([78], dtype=torch.int64, device="cuda")
    claims = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)
    claims[::5] = V - 1
    claims[1::5] = 0

    def score(a, b, call):
        return call(x[a:b], 0.9, seeds, sid[a:b], pos[a:b], claims[a:b])

    def alone(*a):
        return difr.ipt_score(*a)

    def token(*a):
        return difr.ipt_score(*a, want_token=True, want_rank=True)

    def pair(*a):
        return difr.score_both(*a[:5], a[5], a[5], want_token=True)[1]

    for call in (alone, token):
        whole = score(0, N, call)
        for cuts in ([0, 1000, N], [0, 1024, N]):          # 1000, 1024: three vectors; 1100, 1076: one; 2100: fewer workgroups
            parts = [score(a, b, call) for a, b in zip(cuts, cuts[1:])]
            for k, w in whole.items():
                if w is not None:
                    assert torch.equal(w.view(torch.uint8), torch.cat([p[k] for p in parts]).view(torch.uint8)), (call.__name__, k)
        if call is token:
            for k, w in score(0, N, pair).items():
                if w is not None and k != "logit_rank":
                    assert torch.equal(w.view(torch.uint8), whole[k].view(torch.uint8)), k
