"""Outputs have memory of their own, which the binding takes from torch's allocator: at short and longer lengths of either element size
every output is what the call through the C entry leaves in buffers of the caller's, none overlaps another, writing to one or growing
it leaves the others, and each lives as long as it is held."""
import pytest
import torch

import whole_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("N", [0, 1, 63, 64, 65, 255, 256, 257, 1024, 1025])
@pytest.mark.parametrize("inference", [False, True])
def test_outputs_of_short_and_longer_calls(difr, N, inference):
    g = torch.Generator().manual_seed(N)
    V = 640
    x = torch.randn(N, V, generator=g).to(DEV)
    row = torch.arange(N, dtype=torch.int32).to(DEV)
    seeds = torch.tensor([11], device=DEV)
    c = torch.randint(0, V, (N,), generator=g, dtype=torch.int32).to(DEV)
    at = (0.9, seeds, row * 0, row)
    print("short outputs", N, inference, flush=True)
    want = whole_rows.score_both(x, *at, c, c, want_rank=True, want_token=True, want_log_mass=True) if N else None
    with torch.inference_mode(inference):
        got = difr.score_both(x, *at, c, c, want_rank=True, want_token=True, want_log_mass=True)
        cls = difr.classify(got[0]["margin"], got[0]["logit_rank"], 0.05, 8, V) if N else {}
        pooled = difr.seq_reduce(got[0]["margin"], got[0]["flags"], torch.tensor([0, N], device=DEV), 0.05) if N else {}
    outs = [t for d in (*got, cls, pooled) for t in d.values()]
    spans = sorted((t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in outs if t.numel())
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:])) and all(a % 16 == 0 for a, _ in spans)
    for t in outs:
        assert t.is_contiguous() and t.is_leaf and not t.requires_grad and t.is_inference() == inference and t._base is None
    if not N:
        assert all(t.shape[0] == 0 for d in got for t in d.values())
        return
    for mine, ref in zip(got, want):
        assert set(mine) == set(ref)
        for k in ref:
            assert mine[k].dtype == ref[k].dtype and torch.equal(mine[k].view(torch.uint8), ref[k].view(torch.uint8)), k
    if not inference:
        got[0]["margin"].fill_(7.0)
        side = torch.cuda.Stream()
        got[0]["flags"].record_stream(side)
        assert torch.equal(got[0]["argmax"], want[0]["argmax"]) and torch.equal(got[0]["flags"], want[0]["flags"])
    keep, ref = got[1]["dist"], want[1]["dist"]
    del got, cls, pooled, outs
    for _ in range(8):                               # new outputs do not land where one that is held lives
        difr.score_both(x, 1.3, seeds, row * 0, row, None, None)
    assert torch.equal(keep.view(torch.uint8), ref.view(torch.uint8))


@pytest.mark.parametrize("N", [1, 64, 256])
def test_an_output_that_grows_leaves_the_others(difr, N):
    """In-place growth, and an operation that resizes its out argument, end in memory of the tensor's own; an output that is kept or
    saved holds its own bytes."""
    V = 512
    x = torch.randn(N, V, generator=torch.Generator().manual_seed(N)).to(DEV)
    row = torch.arange(N, dtype=torch.int32, device=DEV)
    c = (row * 7) % V
    print("short outputs, growing", N, flush=True)
    got = difr.score_both(x, 0.9, torch.tensor([11], device=DEV), row * 0, row, c, c, want_rank=True, want_log_mass=True)
    outs = [(i, k, t) for i, d in enumerate(got) for k, t in d.items()]
    for _, k, t in outs:
        assert t.untyped_storage().nbytes() == t.numel() * t.element_size() and t.storage_offset() == 0, k
    before = {(i, k): t.clone() for i, k, t in outs}
    grown = got[0]["margin"].resize_(4 * N)
    grown.fill_(7.0)
    torch.add(torch.ones(2 * N, device=DEV), 1.0, out=got[1]["cdf_lo"].resize_(0))
    for i, k, t in outs:
        if (i, k) not in ((0, "margin"), (1, "cdf_lo")):
            assert torch.equal(t.view(torch.uint8), before[i, k].view(torch.uint8)), k
    assert bool((grown == 7.0).all()) and bool((got[1]["cdf_lo"] == 2.0).all())


def test_outputs_under_a_dispatch_mode_and_filled(difr):
    """A mode that watches allocations sees those of the outputs, and with deterministic algorithms the results are the same."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        n = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.n += "empty" in str(func)
            return func(*args, **(kwargs or {}))

    x = torch.randn(8, 512, generator=torch.Generator().manual_seed(2)).to(DEV)
    row = torch.arange(8, dtype=torch.int32, device=DEV)
    at = (x, 0.9, torch.tensor([11], device=DEV), row * 0, row, row)
    print("short outputs, watched", flush=True)
    want = difr.gumbel_score(*at)
    with Seen() as seen:
        got = difr.gumbel_score(*at)
    assert seen.n >= len(got)
    torch.use_deterministic_algorithms(True)
    try:
        filled = difr.gumbel_score(*at)
    finally:
        torch.use_deterministic_algorithms(False)
    for k in want:
        assert torch.equal(got[k].view(torch.uint8), want[k].view(torch.uint8)) and torch.equal(filled[k].view(torch.uint8), want[k].view(torch.uint8)), k
