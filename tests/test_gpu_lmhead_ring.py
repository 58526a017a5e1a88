"""The small-batch LM-head kernel in its steady state: many slabs per workgroup, so that every LDS stage is refilled while others are
multiplied, in every tile (32, 64 and 128 tokens by 128 and 256 entries), with one and several tiles per range, and with weights
that no cache holds (read past the caches).  Every output of a sample of rows (all of a small batch) against the oracle, with and
without the outputs that have kernels of their own; tolerances of test_gpu_lmhead.py."""
import numpy as np
import pytest
import torch

import oracle
import parity
import test_gpu_lmhead as base

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("N,V,d", [
    (3, 1300, 1024), (33, 1300, 1024), (100, 1300, 1088), (128, 9000, 1536),   # 128-entry tiles, 16 to 24 slabs
    (100, 40000, 512),                                                         # ... two tiles per range: 16 slabs
    (3, 66000, 640), (33, 66000, 704), (100, 66000, 640), (64, 70000, 1024),   # 256-entry tiles, two per range: 20 to 32 slabs
    (20, 70000, 2048), (50, 70000, 2048), (128, 70000, 2048)])                 # 287 MB of weights: 64 slabs, read past the caches
def test_many_slabs(difr, N, V, d):
    wl = base._case(1, N, V, d, T=0.9)
    Wm = wl.weight(DEV)
    Hv, Hp = wl.hidden(DEV)
    seeds, sid, pos = wl.seeds().to(DEV), wl.seq_ids().to(DEV), wl.positions().to(DEV)
    base.say("lmhead ring", N, V, d)
    g0, i0 = difr.lmhead_score(Hp, Wm, wl.temperature, seeds, sid, pos, want_token=True)
    gen = torch.Generator().manual_seed(N + V)
    other = torch.randint(0, V, (N,), generator=gen, dtype=torch.int32).to(DEV)
    k = torch.arange(N, device=DEV)
    cg, ci = torch.where(k % 4 == 1, other, g0["argmax"]), torch.where(k % 4 == 2, other, i0["ipt_token"])
    # the oracle's product takes about a second per 1e9 multiplications
    rows = np.unique(np.linspace(0, N - 1, min(N, max(2, int(1.5e9 // (V * d))))).astype(int))
    at = torch.from_numpy(rows).to(DEV)
    T = np.float32(wl.temperature)
    hs, hsid, hpos = parity.seeds_u64(seeds), sid.cpu().numpy()[rows], parity.positions_u32(pos)[rows]
    hg, hi = cg.cpu().numpy()[rows], ci.cpu().numpy()[rows]
    og, oi, ox = oracle.lmhead_score(base.bits(Hv[at]), base.bits(Wm), T, hs, hsid, hpos, hg, hi, sigma=0.02, want_logits=True)
    first = None
    for opt in (dict(want_rank=True, want_token=True), dict(want_rank=True), dict(want_token=True), {}):
        g, i = difr.lmhead_score(Hv, Wm, wl.temperature, seeds, sid, pos, cg, ci, want_log_mass=True, sigma=0.02, **opt)
        torch.cuda.synchronize()
        g, i = ({k: v[at] for k, v in part.items()} for part in (g, i))
        if "logit_rank" in g:
            base._check_rank(g.pop("logit_rank").cpu().numpy(), ox, hg, V, base.TIE)
        if "ipt_token" in i:
            base._check_token(i.pop("ipt_token").cpu().numpy(), oi, ox, T, hs, hsid, hpos, i["flags"].cpu().numpy())
        parity.compare_gumbel(g, og, tie_rel=base.TIE)
        assert parity.compare_ipt(i, oi, tie_rel=base.TIE, log_mass_sigma=0.02)["log_mass_beyond_bar"] == 0
        first = first or (g, i)
        for a, b in zip(first, (g, i)):           # the variants sum the same logits in the same order
            for key in a:
                if key != "flags":
                    assert torch.equal(a[key].view(torch.int32), b[key].view(torch.int32)), (opt, key)
