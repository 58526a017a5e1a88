"""Small batches, whose rows are shared by several workgroups, against the one-workgroup kernels (whole_rows.py): the Token-DiFR
outputs, ranks and admissible counts bit for bit, the Token-IPT-DiFR sums - formed in another order - to 2e-7 of the CDF (a few
times the 1e-8 that either order is off by, and the fp32 rounding of a value below 1); matches, log-masses and the sampler's token
against the oracle.  Around the smallest vocabulary that is shared, ragged ends, claims in the first and last part, rejected rows, masked parts, a NaN and a
+inf in a later part, and candidate lists that do not fit."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import parity
import whole_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _same(a, b, what):
    for k in a:
        assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), (what, k)


def _near(a, b, what, tol=2e-7):
    for k in a:
        x, y = a[k], b[k]
        if k in ("u", "flags"):
            assert torch.equal(x & ~9, y & ~9) if k == "flags" else torch.equal(x.view(torch.int32), y.view(torch.int32)), (what, k)
        elif k in ("dist", "cdf_lo", "cdf_hi"):
            assert torch.equal(x.isnan(), y.isnan()) and float((x - y).nan_to_num().abs().max()) <= tol, (what, k)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V,N", [(49152, 3), (49153, 24), (65000, 130), (99991, 7), (151936, 24), (151936, 1)])
def test_shared_rows_score_as_whole_rows(difr, dtype, V, N):
    lib = difr.load_library()
    assert lib.difr_split_workspace_bytes(N, V, 0 if dtype == torch.bfloat16 else 1, 0) > 0
    g = torch.Generator().manual_seed(V + N)
    S = min(N, 3)
    x = torch.randn(N, V, generator=g) - 1.1 * torch.log1p(torch.randperm(V, generator=g).float())
    if N >= 7:
        x[1, : V // 2] = -float("inf")            # whole parts without mass
        x[2, ::2] = -float("inf")
        x[4, V - 5] = float("inf")
        x[5] = -float("inf")
        x[5, V - 1] = 0.5
    per = 16 // torch.tensor([], dtype=dtype).element_size()
    buf = torch.zeros(N, -(-V // per) * per, dtype=dtype)
    buf[:, :V] = x.to(dtype)
    if N >= 7:                                    # a NaN with its sign bit clear (one with it set counts as -inf)
        buf.view(torch.int16 if per == 8 else torch.int32)[3, V - 2] = 0x7FC0 if per == 8 else 0x7FC00000
    x = buf.to(DEV)[:, :V]
    seeds = torch.randint(-2 ** 63, 2 ** 63 - 1, (S,), generator=g).to(DEV)
    sid, pos = (torch.arange(N, dtype=torch.int32) % S).to(DEV), torch.arange(N, dtype=torch.int32).to(DEV)
    if N >= 24:
        sid[N - 1] = S
    at = (0.9, seeds, sid, pos)
    honest = difr.gumbel_score(x, *at)["argmax"].clamp(min=0)
    cg = torch.where(torch.arange(N, device=DEV) % 2 == 0, honest, torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV))
    ci = torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV)
    ci[0] = 0
    if N >= 7:
        ci[1], ci[2], cg[3] = V - 1, -1, V
    for delta in (2.5, 12.0):                     # (12: thousands of candidates, more than a part's list holds)
        print("split", dtype, V, N, delta, flush=True)
        ga, ia, ca = difr.score_both_admissible(x, *at, delta, cg, ci)
        wg, wi, wc = whole_rows.score_both_admissible(x, *at, delta, cg, ci)
        two = difr.admissible_count(x, *at, wg["max_score"], delta)
        _same(ga, wg, "admissible")
        _near(ia, wi, "admissible")
        _same(ca, two, "admissible")
        known = wc["count"] >= 0                  # (a whole row's lists may not hold them all)
        assert torch.equal(ca["count"][known], wc["count"][known]) and (delta > 3 or bool(known.any()))
    want_g, want_i = whole_rows.score_both(x, *at, cg, ci, want_rank=True, want_token=True, want_log_mass=True)
    gb, ib = difr.score_both(x, *at, cg, ci, want_rank=True, want_token=True, want_log_mass=True)
    _same(gb, want_g, "both")
    _near(ib, want_i, "both")
    _same({k: ia[k] for k in ia}, {k: ib[k] for k in ia if k != "flags"} | {"flags": ib["flags"] & ~8}, "admissible against both")
    gs = difr.gumbel_score(x, *at, cg, want_rank=True)
    _same(gs, gb, "gumbel")
    si = difr.ipt_score(x, *at, ci, want_token=True, want_log_mass=True, want_rank=True)
    ranks = difr.gumbel_score(x, *at, ci, want_rank=True)["logit_rank"]
    clean = torch.arange(N, device=DEV) != (3 if N >= 7 else N)   # (bit patterns count a NaN as above, values do not)
    assert torch.equal(si.pop("logit_rank")[clean], ranks[clean])
    _same(si, ib, "ipt")
    gp, ip = difr.score_both_peaked(x, *at, cg, ci)
    _same(gp, {k: gb[k] for k in gp}, "peaked")
    _same({k: ip[k] for k in ip if k != "flags"}, {k: ib[k] for k in ip if k != "flags"}, "peaked")
    wg, wi = whole_rows.score_both(x, *at, cg, ci, peaked=True)
    _same(wg, {k: want_g[k] for k in wg}, "peaked, whole rows")
    _same({k: wi[k] for k in wi if k != "flags"}, {k: want_i[k] for k in wi if k != "flags"}, "peaked, whole rows")
    # matches, the sampler's token and the log-mass, of the shared rows and of the whole ones
    ok = ((want_i["flags"] & 4) == 0) & (sid < S)  # (the outputs of a flagged row are unspecified)
    h, T = parity.to_host_logits(x[ok]), float(np.float32(0.9))
    row_args = (T, parity.seeds_u64(seeds), sid[ok].cpu().numpy(), parity.positions_u32(pos[ok]))
    ref = oracle.ipt_score(h, V, *row_args, ci[ok].cpu().numpy(), sigma=0.01)
    for got in (ib, want_i):
        parity.compare_ipt({k: v[ok] for k, v in got.items()}, ref, h, V, row_args, log_mass_sigma=0.01)


def test_capture_and_two_streams(difr):
    """The workspace is the call's own: replays with new inputs and eager work in between, and two streams at once, give what
    an eager call gives."""
    N, V = 24, 65000
    g = torch.Generator().manual_seed(3)
    make = lambda: (torch.randn(N, V, generator=g) * 2.5).to(torch.bfloat16).to(DEV)
    x, inputs = make(), [make() for _ in range(3)]
    seeds = torch.tensor([5, 6], device=DEV)
    sid, pos = (torch.arange(N, device=DEV) % 2).int(), torch.arange(N, device=DEV).int()
    c = torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV)

    def step(logits):
        return [t for part in difr.score_both(logits, 0.9, seeds, sid, pos, c, c, want_rank=True, want_token=True)
                for t in part.values()]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(x)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = step(x)
    for other in inputs:
        x.copy_(other)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in captured]
        eager = step(x)
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, eager))
    want = [step(i) for i in inputs[:2]]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = [[], []]
    for _ in range(4):
        for k, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[k].append(step(inputs[k]))
    torch.cuda.synchronize()
    for k in range(2):
        for r in got[k]:
            assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(r, want[k]))


def test_what_difr_score_split_refuses(difr):
    from paper_2511_02620_amd import binding as B
    lib = difr.load_library()
    assert lib.difr_split_workspace_bytes(0, 151936, 0, 0) == 0 and lib.difr_split_workspace_bytes(24, 151936, 2, 0) == 0
    assert lib.difr_split_workspace_bytes(24, 8192, 0, 0) == 0 and lib.difr_split_workspace_bytes(16384, 151936, 0, 0) == 0
    N, V = 4, 65536
    x = torch.zeros(N, V, dtype=torch.bfloat16, device=DEV)
    i = torch.zeros(N, dtype=torch.int32, device=DEV)
    r, _, dev = B._rows(x, None, 1.0, torch.zeros(1, dtype=torch.int64, device=DEV), i, i, i, None)
    need = lib.difr_split_workspace_bytes(N, V, 0, 1)
    buf = torch.zeros(max(need, 4096) + 8, dtype=torch.uint8, device=DEV)
    p = buf.data_ptr()

    def call(ws=p, n=need, **kw):
        o = B._Scores(**kw)
        return lib.difr_score_split(C.byref(r), i.data_ptr(), C.byref(o), ws, n, None)
    full = dict(margin=p, argmax=p, flags_gumbel=p, dist=p, flags_ipt=p)
    NULL, SHAPE, ALIGN, ARG = 1, 2, 5, 8
    assert call() == NULL and call(margin=p) == NULL and call(dist=p) == NULL
    assert call(n=lib.difr_split_workspace_bytes(N, V, 0, 0) - 1, **full) == SHAPE and call(ws=None, **full) == NULL
    assert call(ws=p + 4, **full) == ALIGN and call(log_mass=p, sigma=0.0, **full) == ARG
    assert call(count=p, delta=-1.0, **full) == ARG and call(count=p, delta=1.0, ipt_token=p, **full) == ARG
    assert call(count=p, delta=1.0, dist=p, flags_ipt=p) == NULL and call(rank_ipt=p, **full) == ARG
    torch.cuda.synchronize()
    assert int(buf.sum()) == 0


@pytest.mark.parametrize("N,shared", [(320, True), (321, False)])
def test_peaked_rows_are_shared_up_to_a_line(difr, N, shared):
    """Beyond some rows the peaked kernel is the faster one for them: the call then gives its bits, below the line those of
    difr_score_both on shared rows."""
    V = 151936
    g = torch.Generator(device=DEV).manual_seed(N)
    x = torch.empty(N, V, dtype=torch.bfloat16, device=DEV)
    x.copy_(-3.0 * torch.log1p(torch.randperm(V, generator=g, device=DEV).float()) + torch.randn(N, V, generator=g, device=DEV))
    seeds = torch.tensor([5, 6], device=DEV)
    sid, pos = (torch.arange(N, device=DEV) % 2).int(), torch.arange(N, device=DEV).int()
    c = torch.randint(0, V, (N,), generator=g, device=DEV, dtype=torch.int32)
    assert whole_rows.is_shared(x)
    got = difr.score_both_peaked(x, 0.6, seeds, sid, pos, c, c)
    whole = whole_rows.score_both(x, 0.6, seeds, sid, pos, c, c, peaked=True)
    _same(got[0], whole[0], "peaked")
    # (one token carries most of such a row; its exponent lies up to 64 above its thread's reference, where fp32 is good to 1.9e-6
    # in the exponent and 1.3e-6 in the mass, on either side of the comparison)
    _near(got[1], whole[1], "peaked", 2.6e-6)
    bits = lambda t: t.view(torch.int32)
    assert torch.equal(bits(got[1]["cdf_lo"]), bits(whole[1]["cdf_lo"])) == (not shared)
    both = difr.score_both(x, 0.6, seeds, sid, pos, c, c)
    assert torch.equal(bits(got[1]["cdf_lo"]), bits(both[1]["cdf_lo"])) == shared
