"""difr_lmhead_score at the sizes where its work split changes: token counts around the merge kernel's groups of 8 and the
token tiles (32, 64, 128 and 256 rows), vocabularies around a vocabulary tile (128 and 256 entries) and with more ranges than the merge has threads per token.  Every
row, every output, against the oracle, with the tolerances of test_gpu_lmhead.py (whose comparison helpers this uses)."""
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


@pytest.mark.parametrize("N,V,d", [(1, 1, 64), (1, 9000, 64), (7, 255, 64), (8, 256, 128), (9, 257, 64), (17, 8500, 128),
                                   (64, 1300, 192), (3, 128, 64), (33, 129, 64), (63, 385, 64), (64, 70000, 64), (65, 256, 128),
                                   (66, 513, 64), (32, 257, 64), (32, 70000, 64), (2, 66000, 128), (100, 70000, 64), (128, 1300, 192), (129, 1300, 64)])
def test_every_output_at_split_edges(difr, N, V, d):
    wl = base._case(1, N, V, d, T=0.9)
    Wm = wl.weight(DEV)
    Hv, Hp = wl.hidden(DEV)
    seeds, sid, pos = wl.seeds().to(DEV), wl.seq_ids().to(DEV), wl.positions().to(DEV)
    base.say("lmhead shape", N, V, d)
    hs, hsid, hpos = parity.seeds_u64(seeds), sid.cpu().numpy(), parity.positions_u32(pos)
    T = np.float32(wl.temperature)
    og0, oi0 = oracle.lmhead_score(base.bits(Hp), base.bits(Wm), T, hs, hsid, hpos, None, None)
    gen = torch.Generator().manual_seed(N + V)
    other = torch.randint(0, V, (N,), generator=gen, dtype=torch.int32)
    k = torch.arange(N)
    cg = torch.where(k % 4 == 1, other, torch.from_numpy(og0["argmax"].copy())).to(DEV)
    ci = torch.where(k % 4 == 2, other, torch.from_numpy(oi0["ipt_token"].copy())).to(DEV)
    for claims_g, claims_i in ((cg, ci), (None, None)):
        g, i = difr.lmhead_score(Hv, Wm, wl.temperature, seeds, sid, pos, claims_g, claims_i, want_rank=True,
                                 want_log_mass=True, want_token=True, sigma=0.02)
        plain = difr.lmhead_score(Hv, Wm, wl.temperature, seeds, sid, pos, claims_g, claims_i)
        torch.cuda.synchronize()
        hg, hi = (None if c is None else c.cpu().numpy() for c in (claims_g, claims_i))
        og, oi, ox = oracle.lmhead_score(base.bits(Hv), base.bits(Wm), T, hs, hsid, hpos, hg, hi, sigma=0.02, want_logits=True)
        base._check_rank(g.pop("logit_rank").cpu().numpy(), ox, hg, V, base.TIE)
        base._check_token(i.pop("ipt_token").cpu().numpy(), oi, ox, T, hs, hsid, hpos, i["flags"].cpu().numpy())
        parity.compare_gumbel(g, og, tie_rel=base.TIE)
        assert parity.compare_ipt(i, oi, tie_rel=base.TIE, log_mass_sigma=0.02)["log_mass_beyond_bar"] == 0
        # without the optional outputs the same scores
        for a, b, keys in ((plain[0], g, ("margin", "argmax", "max_score", "claimed_score")),
                           (plain[1], i, ("cdf_lo", "cdf_hi", "dist", "u"))):
            for key in keys:
                x, y = a[key].cpu().numpy(), b[key].cpu().numpy()
                np.testing.assert_allclose(x, y, rtol=0, atol=0 if key in ("argmax", "u") else parity.ABS_TOL, equal_nan=True)
