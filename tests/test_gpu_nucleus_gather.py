"""Nuclei whose cut falls among entries above everything that has been looked at, so that they are gathered at once: one
entry, as many as one thread each takes and one more (two ways of sorting), and more than the buffer holds (the search then
goes on).  bf16 rows of ordinary values are counted instead; those of the kind "searched" have so few values where they are looked at that
they are not, which is asserted.  Against the oracle with the bounds of test_gpu_nucleus.py."""
import pytest
import torch

import nucleus_look
import test_gpu_nucleus as base

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _few_values_where_looked_at(x, V):
    """Puts one value where a bf16 row is looked at, and -10 at one place: a span of bins with one entry in the top one."""
    seen = torch.zeros(V // 8, 8, dtype=torch.bool)
    seen[nucleus_look.looked_at(V)] = True
    seen = seen.view(-1)
    x[:, seen] = -20.0
    x[:, 3] = -10.0
    return (~seen).nonzero().squeeze(1)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32, "searched"])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 512, 2048, 2049, 6000])
def test_heavy_entries_beyond_the_first_round(difr, dtype, n):
    N, V, S = 6, 20008, 2
    g = torch.Generator().manual_seed(n)
    x = -20 - torch.rand(N, V, generator=g)
    x[:, 100] = -10.0                                  # the first round's largest: a span of bins, one entry in the top one
    free = _few_values_where_looked_at(x, V) if dtype == "searched" else torch.arange(2048, V)
    for r in range(N):
        at = free[torch.randperm(len(free), generator=g)[:n]]
        x[r, at] = 4 + 5 * torch.rand(n, generator=g)
    x[4] = x[4].round()                                # ties
    if dtype == "searched":
        assert not nucleus_look.counted_first(x.bfloat16(), V, 0.8).any()
    x = x.to(torch.bfloat16 if dtype == "searched" else dtype).to(DEV)
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    claims = x.argmax(1).int()
    claims[1], claims[2] = V - 1, 0
    for p in (0.5, 0.93):
        print("nucleus gather", dtype, n, p, flush=True)
        base._compare(difr, x, V, 0.8, seeds, sid, pos, claims, p)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32, "searched"])
@pytest.mark.parametrize("n", [2048, 2049, 6000])
def test_heavy_entries_that_the_sample_misses(difr, dtype, n):
    """The sample that decides whether a bracket is gathered at once is every step-th vector: heavy entries between its vectors
    are gathered up to what the buffer holds, and beyond it the search goes on."""
    N, V, S = 4, 20008, 2
    per = 4 if dtype == torch.float32 else 8
    nvec = -(-V // per)
    step = nvec // 256
    g = torch.Generator().manual_seed(n)
    x = -20 - torch.rand(N, V, generator=g)
    x[:, 100] = -10.0
    vec = torch.arange(V) // per
    free = (vec % step != 0) & (vec >= 256) & (torch.arange(V) != 100)
    if dtype == "searched":
        unseen = torch.zeros(V, dtype=torch.bool)
        unseen[_few_values_where_looked_at(x, V)] = True
        free &= unseen
    free = free.nonzero().squeeze(1)
    for r in range(N):
        x[r, free[torch.randperm(len(free), generator=g)[:n]]] = 4 + 5 * torch.rand(n, generator=g)
    x[3] = x[3].round()
    if dtype == "searched":
        assert not nucleus_look.counted_first(x.bfloat16(), V, 0.8).any()
    x = x.to(torch.bfloat16 if dtype == "searched" else dtype).to(DEV)
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    claims = x.argmax(1).int()
    claims[1], claims[2] = V - 1, 0
    for p in (0.5, 0.93):
        print("nucleus gather, unseen", dtype, n, p, flush=True)
        base._compare(difr, x, V, 0.8, seeds, sid, pos, claims, p)
