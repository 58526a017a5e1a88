"""Entries masked with a very low finite logit (the type's lowest value, as attention-style masks write it, or -1e4 ... -1e10)
have no mass and change nothing else, wherever they lie: in the first vectors of a row's threads, from which the softmax sums
take their exponent reference, in whole parts of a row that several workgroups share, around a claim.  Both scores of every row
against the oracle."""
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


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [5000, 65000])    # one workgroup per row, and rows that are shared
@pytest.mark.parametrize("T", [0.6, 1.0, 2.3])
def test_low_masks_have_no_mass(difr, dtype, V, T):
    N, S = 8, 2
    T = float(np.float32(T))
    g = torch.Generator().manual_seed(V)
    base = torch.randn(N, V, generator=g) * 2
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g)
    sid, pos = torch.arange(N, dtype=torch.int32) % S, torch.arange(N, dtype=torch.int32)
    for low in (torch.finfo(dtype).min, -1e10, -3e9, -1e9, -1e4):
        x = base.clone()
        x[0, V // 2:] = low
        x[1, : V // 2] = low
        x[2, : 2048] = low                      # every thread's first vector
        x[3, V - 300:] = low                    # a padded vocabulary
        x[4, 1::2] = low
        x[5, 3:] = low                          # three entries left, all at the start ...
        x[6, : V - 3] = low                     # ... and at the end
        x[7, V // 3: V // 3 + 9000] = low
        x = x.to(dtype)
        claims = x.float().argmax(1).int()
        claims[0], claims[1], claims[3] = V - 1, 0, V // 2
        h = parity.to_host_logits(x)
        at = (T, parity.seeds_u64(seeds), sid.numpy(), parity.positions_u32(pos))
        og, oi = oracle.gumbel_score(h, V, *at, claims.numpy()), oracle.ipt_score(h, V, *at, claims.numpy())
        print("low masks", dtype, V, T, low, flush=True)
        gg, gi = difr.score_both(x.to(DEV), T, seeds.to(DEV), sid.to(DEV), pos.to(DEV), claims.to(DEV), claims.to(DEV), want_token=True)
        assert not (gi["flags"] & 4).any(), (low, gi["flags"])
        # a masked claim's margin is some 4e3 and more, where fp32 values lie 5e-4 apart: those two rows are left out
        keep = np.abs(og["margin"]) < 1e3
        assert parity.compare_ipt(gi, oi, h, V, at)["rows"] == N
        parity.compare_gumbel({k: v.cpu()[torch.from_numpy(keep)] for k, v in gg.items()}, {k: v[keep] for k, v in og.items()})
        alone = difr.ipt_score(x.to(DEV), T, seeds.to(DEV), sid.to(DEV), pos.to(DEV), claims.to(DEV), want_token=True)
        for k in gi:
            assert torch.equal(gi[k].view(torch.uint8), alone[k].view(torch.uint8)), k
