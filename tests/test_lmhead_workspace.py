"""The workspace of difr_lmhead_score: one sized for a batch of up to 256 tokens serves every smaller one, and what a range per 256
vocabulary entries (256 at most) takes is enough for any batch of up to 256 tokens - the vocabulary is then cut into fewer ranges,
with the same results."""
import ctypes as C

import pytest
import torch

import paper_2511_02620_amd as difr
from paper_2511_02620_amd import binding as B

SHAPE, UNSUPPORTED = 2, 7
VOCABS = (1, 255, 4000, 16000, 32000, 50257, 65536, 65537, 100000, 151936)


def _least(N, V, token=False):
    n_vt = -(-V // 256)
    return N * min(256, n_vt) * 32 + 16 * N + 64 + (16 * N * n_vt + 16 * N if token else 0)


@pytest.mark.parametrize("V", VOCABS)
@pytest.mark.parametrize("token", [False, True])
def test_named_size_does_not_fall(V, token):
    sizes = [difr.lmhead_workspace_bytes(N, V, 4096, want_token=token) for N in range(1, 257)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="the accepted calls would launch on made-up pointers")
@pytest.mark.parametrize("V", VOCABS)
@pytest.mark.parametrize("token", [False, True])
def test_which_sizes_are_taken(V, token):
    lib, fake = difr.load_library(), 0x1000
    r = B._LmHead()
    r.hidden, r.weight, r.V, r.d, r.ldh, r.ldw, r.temperature, r.S = fake, fake, V, 64, 64, 64, 1.0, 1
    r.seeds, r.seq_ids, r.positions = fake, fake, fake

    def call(N, ws_bytes):
        r.N = N
        return lib.difr_lmhead_score(C.byref(r), fake, fake, None, None, fake, None, fake, None, None, None,
                                     fake if token else None, 0.01, 1e-30, None, fake, fake, ws_bytes, None)
    for N in (1, 3, 32, 33, 64, 65, 100, 127, 128, 129, 200, 256):
        assert call(N, _least(N, V, token)) == UNSUPPORTED, N           # (accepted: it ends at the missing device)
        for larger in (N, N + 1, 129, 255, 256):
            if N <= larger <= 256:
                assert call(N, difr.lmhead_workspace_bytes(larger, V, 64, want_token=token)) == UNSUPPORTED, (N, larger)
        if N > 128 or V <= 128:
            assert call(N, _least(N, V, token) - 1) == SHAPE, N
        assert call(N, 32 * N) == SHAPE


@pytest.mark.gpu
@pytest.mark.parametrize("N,V", [(3, 4000), (64, 16000), (128, 32000), (33, 65536)])
def test_fewer_ranges_give_the_same_scores(N, V):
    dev, d = "cuda:0", 128
    g = torch.Generator(device=dev).manual_seed(N)
    h = torch.randn(N, d, generator=g, device=dev).bfloat16()
    w = (torch.randn(V, d, generator=g, device=dev) / d ** 0.5).bfloat16()
    seeds = torch.arange(1, 4, device=dev)
    at = (h, w, 0.9, seeds, (torch.arange(N, device=dev) % 3).int(), torch.arange(N, device=dev).int())
    c = torch.randint(0, V, (N,), generator=g, device=dev).int()
    for token in (False, True):
        opt = dict(want_rank=True, want_log_mass=True, want_token=token)
        print("lmhead workspace", N, V, token, flush=True)
        want = difr.lmhead_score(*at, c, c, **opt)
        small = torch.zeros(_least(N, V, token) + 4096, dtype=torch.uint8, device=dev)
        got = difr.lmhead_score(*at, c, c, workspace=small[:_least(N, V, token)], **opt)
        assert int(small[_least(N, V, token):].sum()) == 0
        for a, b in zip(want, got):
            for k in a:
                if k in ("dist", "cdf_lo", "cdf_hi", "log_mass"):
                    # fp64 sums of the same terms, grouped differently: the last bit of the fp32 result (log_mass: of up to 70)
                    assert float((a[k] - b[k]).abs().max()) <= (8e-6 if k == "log_mass" else 6e-8), k
                else:
                    assert torch.equal(a[k], b[k]), k
