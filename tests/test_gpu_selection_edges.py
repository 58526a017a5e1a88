"""The streaming selections where they change their way (csrc/topn.hpp, csrc/likelihood.hip, csrc/ipt_filtered.hip): sizes at which the
first thresholds are formed from 64, 128 or 256 keys and the buffers grow, rows too short for the rounds spread over them, and rows
whose entries share the keys' bits (masked, coarse, constant) or rise from round to round.  Active set, threshold and estimate against
the oracle, the filtered interval against the definition in 64 bits."""
import pytest
import torch

import paper_2511_02620_amd as difr
from test_gpu_likelihood import _compare

pytestmark = pytest.mark.gpu
DEV = "cuda"

SIZES = [(64, 64), (16, 65), (65, 16), (32, 33), (100, 101), (128, 128), (129, 100), (256, 256)]  # (s, top_k)
ROWS = [("random", 2048 * 9), ("random", 2040), ("masked", 2048 * 4 + 8), ("late", 2048 * 5), ("coarse", 2048 * 4), ("constant", 4096),
        ("rising", 2048 * 18)]


def _logits(order, N, V, dtype, g):
    x = 2.5 * torch.randn(N, V, generator=g, device=DEV)
    if order == "masked":                                       # twenty entries of the row are not masked
        keep = torch.rand(N, V, generator=g, device=DEV).topk(20, dim=1).indices
        x = torch.full_like(x, -torch.inf).scatter_(1, keep, x.gather(1, keep))
    elif order == "late":                                       # nothing in the first round
        x[:, :2048] = -torch.inf
    elif order == "coarse":
        x = (x / 2).round()
    elif order == "constant":
        x = torch.ones_like(x)
    elif order == "rising":                                     # every round lies above the ones before it
        x += torch.arange(V, device=DEV) // 1024
    return x.to(dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("s,k", SIZES)
@pytest.mark.parametrize("order,V", ROWS)
def test_selections_at_their_edges(dtype, s, k, order, V):
    N, T, p = 6, 0.9, 0.95
    g = torch.Generator(device=DEV).manual_seed(V + s + k)
    x = _logits(order, N, V, dtype, g)
    sid = torch.zeros(N, dtype=torch.int32, device=DEV)
    pos = torch.arange(N, dtype=torch.int32, device=DEV)
    seeds = torch.tensor([11 + s], dtype=torch.int64, device=DEV)
    claims = x.float().argmax(dim=1).int()
    _compare(difr, x, V, T, seeds, sid, pos, claims, k, p, s, 0.4)

    out = difr.ipt_score_filtered(x, T, seeds, sid, pos, claims, top_k=k, top_p=p)
    val, idx = x.double().sort(dim=1, descending=True, stable=True)
    val, idx = val[:, :k], idx[:, :k]
    e = ((val - val[:, :1]) / torch.tensor(T, dtype=torch.float32).double().item()).exp()
    before = e.cumsum(1) - e
    inside = before < torch.tensor(p, dtype=torch.float32).double().item() * e.sum(1, keepdim=True)
    kept = inside.sum(1)
    # the cut may fall on either side of a sum that ends within rounding of top_p: 256 terms in 64 bits, 1e-13 of the sum at most
    near = ((before / e.sum(1, keepdim=True) - torch.tensor(p, dtype=torch.float32).double().item()).abs() < 1e-12).any(1)
    assert torch.equal(out["kept"].long()[~near], kept[~near])
    e = torch.where(inside, e, 0.0)
    own = (idx == claims.long().unsqueeze(1)) & inside
    width = (torch.where(own, e, 0.0).sum(1) / e.sum(1))
    below = torch.where(inside & (idx < claims.long().unsqueeze(1)), e, 0.0).sum(1) / e.sum(1)
    # interval ends are fp32 roundings (6e-8) of fp64 quotients
    assert ((out["cdf_lo"].double() - below).abs()[~near] < 1e-7).all()
    assert ((out["cdf_hi"].double() - below - width).abs()[~near] < 1e-7).all()
