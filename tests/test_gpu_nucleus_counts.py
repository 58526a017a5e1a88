"""bf16 nuclei that one read with a counter per logit value decides, and rows that it leaves to the search: values at the edges of
the counted range (2^-10, 127.5, 128, -128), entries around zero, masked entries, a cut on a shared counter, rows of few values,
rows shorter than a round and with ragged ends.  Against the oracle with the bounds of test_gpu_nucleus.py."""
import pytest
import torch

import test_gpu_nucleus as base

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _rows(kind, N, V, g):
    x = torch.randn(N, V, generator=g) * 2
    edge = torch.randperm(V, generator=g)
    if kind == "shifted":
        x -= 11
    elif kind == "edges":  # the lowest and highest counted values and their neighbours, either sign
        e = torch.tensor([2.0 ** -10, -2.0 ** -10, 2.0 ** -10 * (1 + 2.0 ** -7), -2.0 ** -10 * (1 + 2.0 ** -7), -127.5, -127.0])
        x[:, edge[:min(V, 600)]] = e[torch.arange(min(V, 600)) % 6]
    elif kind == "large":  # rows 0 and 1 hold a value of 127.5 and 128, the others neither
        x += 100
        x[0, edge[0]], x[1, edge[0]] = 127.5, 128.0
    elif kind == "low":    # entries of -128 and less, with mass and without
        x -= 130
        x[::2, edge[0]] = 5.0
    elif kind == "zeros":  # hundreds of zeros and values around them: the cut may lie among them
        x = x * 2.0 ** -9
        x[:, edge[:V // 3]] = 0.0
    elif kind == "masked":
        x[:, edge[V // 20 + 1:]] = -float("inf")
        x[1, edge[V // 20 + 1:]] = -3.3895314e38
        x[2] = -float("inf")
        x[2, edge[0]] = -3.0
    elif kind == "few":    # rows of few values
        x = x.round()
        x[1] = 1.5
        x[2] = 0.0
    return x.bfloat16()


@pytest.mark.parametrize("V", [1, 7, 8, 1000, 2047, 2048, 2056, 4099, 20004])
@pytest.mark.parametrize("kind", ["plain", "shifted", "edges", "large", "low", "zeros", "masked", "few"])
def test_counted_rows(difr, kind, V):
    N, S = 6, 2
    g = torch.Generator().manual_seed(V)
    x = torch.empty(N, -(-V // 8) * 8, dtype=torch.bfloat16)
    x[:, V:] = float("nan")                        # never read into a result
    x[:, :V] = _rows(kind, N, V, g)
    x = x.to(DEV)[:, :V]
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    claims = x.float().nan_to_num(-1e30).argmax(1).int()
    claims[1], claims[2], claims[3] = V - 1, 0, V // 2
    for p, T in ((0.93, 0.8), (0.5, 1.3)):
        print("nucleus counts", kind, V, p, flush=True)
        base._compare(difr, x, V, T, seeds, sid, pos, claims, p)


@pytest.mark.parametrize("V", [1, 7, 9, 2047, 2051, 20004, 20008])
def test_low_and_masked_entries_at_high_temperatures(difr, V):
    """Where entries of -128 have mass: rows with -inf only, with one finite entry of -128 and less among them, and with a claim there."""
    N = 6
    g = torch.Generator().manual_seed(V)
    x = torch.empty(N, -(-V // 8) * 8, dtype=torch.bfloat16)
    x[:, V:] = float("nan")
    v = torch.randn(N, V, generator=g) * 2
    low = torch.randperm(V, generator=g)[:max(0, V // 3 - 1)]
    v[1:, low] = -float("inf")
    for r, value in ((2, -128.0), (3, -191.0), (4, -200.0), (5, -3.3895314e38)):
        v[r, low[-1:]] = value
    x[:, :V] = v.bfloat16()
    x = x.to(DEV)[:, :V]
    row = torch.arange(N, dtype=torch.int32, device=DEV)
    claims = v.argmax(1).int()
    if len(low):
        claims[3:5] = int(low[-1])
    for T in (1.2, 2.0, 40.0):
        print("nucleus counts, low entries", V, T, flush=True)
        base._compare(difr, x, V, T, torch.tensor([5], device=DEV), row * 0, row, claims.to(DEV), 0.97)


@pytest.mark.parametrize("V", [1, 8, 2056, 20004])
def test_counted_rows_without_a_distribution(difr, V):
    """A NaN of either sign and +inf: nothing is kept and the row is flagged, with the entry at the row's start, middle and end."""
    bits = [0x7FC0, -1, 0x7F80]
    N = 3 * len(bits)
    x = torch.zeros(N, -(-V // 8) * 8, dtype=torch.bfloat16)
    x[:, :V] = _rows("plain", N, V, torch.Generator().manual_seed(V))
    for r in range(N):
        x.view(torch.int16)[r, (0, V // 2, V - 1)[r // 3]] = bits[r % 3]
    x = x.to(DEV)[:, :V]
    row = torch.arange(N, dtype=torch.int32).to(DEV)
    print("nucleus counts, undefined", V, flush=True)
    out = difr.ipt_score_filtered(x, 0.8, torch.tensor([5]).to(DEV), row * 0, row, row * 0, top_k=0, top_p=0.9, V=V)
    assert (out["flags"] == 4).all() and (out["kept"] == 0).all() and out["dist"].isnan().all()


@pytest.mark.parametrize("temps,scale", [((1.3, 1.5, 4.0, 5.0), 2.0), ((1.3,), 0.02)])
def test_counted_rows_round_trip(difr, temps, scale):
    """A drawn token, scored as a claim, matches with distance 0 and is the token again, over rows whose nuclei hold about 100,000 tokens
    (at a scale of 0.02 with thousands of entries around zero), and a claim is the token exactly where MATCH says so."""
    N, V, p = 4096, 128256, 0.97
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.empty(N, V, dtype=torch.bfloat16, device=DEV)
    for r in range(0, N, 512):
        x[r:r + 512] = (torch.randn(512, V, generator=g, device=DEV) * scale).bfloat16()
    row = torch.arange(N, dtype=torch.int32, device=DEV)
    for T in temps:
        at = (x, T, torch.tensor([5], device=DEV), row * 0, row)
        print("nucleus counts, round trip", T, scale, flush=True)
        drawn = difr.ipt_score_filtered(*at, None, top_k=0, top_p=p, want_token=True)
        tok = drawn["ipt_token"]
        back = difr.ipt_score_filtered(*at, tok, top_k=0, top_p=p, want_token=True)
        missed = int(((back["flags"] & 1) == 0).sum()), int((back["dist"] != 0).sum()), int((back["ipt_token"] != tok).sum())
        print("not matched, at a distance, another token:", missed, "mean kept", float(back["kept"].float().mean()), flush=True)
        assert missed == (0, 0, 0)
        other = torch.where(row % 2 == 0, tok + 1, tok - 1).clamp(0, V - 1)  # a neighbour shares an end of the interval
        near = difr.ipt_score_filtered(*at, other, top_k=0, top_p=p, want_token=True)
        assert torch.equal(near["ipt_token"], tok)
        assert torch.equal((near["flags"] & 1) != 0, other == tok)
