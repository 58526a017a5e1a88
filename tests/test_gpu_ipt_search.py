"""The search for the honest sampler's Token-IPT-DiFR token: marks left in the stream, then a walk from one of them.  Rows
with no full round, the rounds below which a row has no marks and the row is walked from its start, marks that fall on and
beside the end of the full rounds, and more rounds than one batch of the walk, with the mass in the first entries, in the last ones and everywhere, with and without a claim that splits the
stream; every token against the oracle (a token that differs must own an interval within 1e-6 of u: parity.TIE_REL)."""
import numpy as np
import pytest
import torch

import oracle
import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype,rounds,extra", [
    (dt, r, e) for dt in (torch.bfloat16, torch.float32)
    for r, e in ((0, 1), (0, 9), (1, -1), (1, 0), (1, 1), (5, 0), (6, 0), (6, 1), (7, -1), (7, 8), (12, 0), (13, 9), (15, 9), (16, -1), (16, 0),
                 (16, 1), (18, 0), (50, 1021))])
def test_sampled_token_is_the_oracles(difr, dtype, rounds, extra):
    per = 256 * 16 // torch.tensor([], dtype=dtype).element_size()
    V, N, S = rounds * per + extra, 24, 4
    g = torch.Generator().manual_seed(1000 * rounds + extra + 7)
    x = torch.randn(N, V, generator=g) * 2
    x[0:4, : max(1, V // 50)] += 12                 # the mass at the row's start ...
    x[4:8, -max(1, V // 50):] += 12                 # ... at its end ...
    x[8:12, torch.randint(0, V, (1,), generator=g)] += 30   # ... in one entry
    x[12, 1::2] = -float("inf")
    x[13, : V // 2] = -float("inf")
    x = x.to(dtype)
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g)
    sid, pos = torch.arange(N, dtype=torch.int32) % S, torch.arange(N, dtype=torch.int32)
    claim = torch.randint(0, V, (N,), generator=g, dtype=torch.int32)
    claim[1::4] = V - 1
    claim[2::4] = 0
    T = float(np.float32(0.9))
    h = parity.to_host_logits(x)
    at = (T, parity.seeds_u64(seeds), sid.numpy(), parity.positions_u32(pos))
    dev = (T, seeds.to(DEV), sid.to(DEV), pos.to(DEV))
    for c in (None, claim):
        print("ipt search", dtype, V, "no claims" if c is None else "claims", flush=True)
        ref = oracle.ipt_score(h, V, *at, None if c is None else c.numpy())
        got = difr.ipt_score(x.to(DEV), *dev, None if c is None else c.to(DEV), want_token=True)
        parity.compare_ipt(got, ref, h, V, at)
        both = difr.score_both(x.to(DEV), *dev, None, None if c is None else c.to(DEV), want_token=True)[1]
        for k in got:
            assert torch.equal(got[k].view(torch.uint8), both[k].view(torch.uint8)), k
