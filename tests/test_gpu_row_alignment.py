"""Rows that start at any element: packed rows of an odd vocabulary, at every offset from a 16-byte boundary, must score as
the same rows do in a padded, aligned buffer - bit for bit, since the same kernels read them -, around one vector, one
round of 256 vectors and the ragged end, at lengths at which several workgroups share a row, with the packed buffer ending at the
last entry of the last row."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _equal(a, b, what):
    for k in a:
        x, y = a[k].cpu().contiguous().view(torch.uint8), b[k].cpu().contiguous().view(torch.uint8)
        assert torch.equal(x, y), "%s: %s" % (what, k)


@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, v) for v in (1, 7, 9, 2047, 2049, 2063, 4099, 20011)] +
                         [(torch.float32, v) for v in (1, 3, 5, 1023, 1025, 4099)] +
                         [(dt, v) for dt in (torch.bfloat16, torch.float32) for v in (49153, 99991)])
def test_packed_rows_score_as_aligned_rows(difr, dtype, V):
    N, S, per = 9, 3, 16 // torch.tensor([], dtype=dtype).element_size()
    g = torch.Generator().manual_seed(V)
    x = (torch.randn(N, V, generator=g) * 2 - 1.1 * torch.log1p(torch.randperm(V, generator=g).float())).to(dtype)
    x[4, ::3] = -float("inf")
    pad = torch.zeros(N, -(-V // per) * per, dtype=dtype)
    pad[:, :V] = x
    pad = pad.to(DEV)[:, :V]
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    at = (0.8, seeds, sid, pos)
    honest = difr.gumbel_score(pad, *at)["argmax"]
    cg = torch.where(torch.arange(N, device=DEV) % 2 == 0, honest, torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV))
    ci = torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV)
    ci[0], cg[1], ci[2] = V - 1, -1, V
    opt = dict(want_rank=True, want_token=True, want_log_mass=True)
    want = difr.score_both(pad, *at, cg, ci, **opt)
    for offset in range(per):
        print("row alignment", dtype, V, offset, flush=True)
        buf = torch.empty(N * V + offset, dtype=dtype, device=DEV)
        packed = buf[offset:].view(N, V)
        packed.copy_(pad)
        for i, part in enumerate(difr.score_both(packed, *at, cg, ci, **opt)):
            _equal(part, want[i], "score_both offset %d" % offset)
        _equal(difr.gumbel_score(packed, *at, cg, want_rank=True), want[0], "gumbel_score offset %d" % offset)
        _equal(difr.ipt_score(packed, *at, ci, want_token=True, want_log_mass=True), want[1], "ipt_score offset %d" % offset)
        peaked = difr.score_both_peaked(packed, *at, cg, ci, want_token=True, want_log_mass=True)
        _equal(peaked[0], {k: want[0][k] for k in peaked[0]}, "score_both_peaked offset %d" % offset)
        _equal(peaked[1], want[1], "score_both_peaked offset %d" % offset)
        full = difr.gumbel_score(packed, *at, cg, unfiltered=True, want_rank=True)
        _equal(full, want[0], "unfiltered offset %d" % offset)
        _equal(difr.admissible_count(packed, *at, want[0]["max_score"], 2.0),
               difr.admissible_count(pad, *at, want[0]["max_score"], 2.0), "admissible_count offset %d" % offset)
