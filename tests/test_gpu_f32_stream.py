"""The fp32 stream of Token-DiFR, whose gates look at the largest of four logits and which keeps two vectors in flight: rows of 0 to 4 and of
more full rounds (either end of the three-fold loop), NaNs of either sign and infinities at each of the four places of a vector,
against the kernel that evaluates every entry (bit for bit), alone and beside Token-IPT-DiFR, with the bound rising and fixed."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("V", [1, 1023, 1024, 1025, 2048, 3071, 3072, 4100, 5121, 20003])
@pytest.mark.parametrize("shift", [0.0, 40.0, -40.0])
def test_fp32_stream(difr, V, shift):
    N = 16
    g = torch.Generator().manual_seed(V)
    x = torch.randn(N, V, generator=g) * 3 + shift
    at = max(0, V // 2 // 4 * 4 - 8)
    for k in range(4):                              # one place of a vector each
        v = min(V - 1, at + k)
        x[4, v] = float("nan") if k == 0 else x[4, v]
        x[5 + k, v] = -float("nan") if k & 1 else float("nan")
        x[9, v] = -float("inf")
        x[10, v] = float("inf") if k == 3 else -float("inf")
    x[11] = -float("inf")
    x[11, V - 1] = -3.0
    x = x.to(DEV)
    seeds = torch.tensor([3, -7], device=DEV)
    sid, pos = (torch.arange(N, device=DEV) % 2).int(), torch.arange(N, device=DEV).int()
    claim = torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV)
    print("fp32 stream", V, shift, flush=True)
    want = difr.gumbel_score(x, 0.8, seeds, sid, pos, claim, want_rank=True, unfiltered=True)
    for got in (difr.gumbel_score(x, 0.8, seeds, sid, pos, claim, want_rank=True), difr.gumbel_score(x, 0.8, seeds, sid, pos, claim),
                difr.score_both(x, 0.8, seeds, sid, pos, claim, claim, want_rank=True)[0],
                difr.score_both_peaked(x, 0.8, seeds, sid, pos, claim, claim)[0]):
        fine = (want["flags"] & 4) == 0             # (the scores of a flagged row are unspecified)
        assert torch.equal(got["flags"] & 4, want["flags"] & 4)
        for k in got:
            assert torch.equal(got[k][fine].view(torch.uint8), want[k][fine].view(torch.uint8)), k
    fine = ((want["flags"] & 4) == 0) & want["max_score"].isfinite()
    two = difr.admissible_count(x, 0.8, seeds, sid, pos, want["max_score"], 2.0)["count"]
    one = difr.score_both_admissible(x, 0.8, seeds, sid, pos, 2.0, claim, claim)[2]["count"] if V % 4 == 0 else two
    fine &= one >= 0                                # (-1: a random claim's bound let more candidates through than the lists hold)
    assert torch.equal(one[fine], two[fine]) and bool((one >= 0).any())
