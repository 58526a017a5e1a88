"""bf16 nuclei: whether a row is counted in one read or searched for by passes shows in its time.  Rows that differ in nothing that
should decide it - a ragged end, a mask - take about as long as each other, or one light read longer.  Results are compared in the other nucleus tests."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 1024


@pytest.fixture(scope="module")
def difr():
    import paper_2511_02620_amd as m
    m.load_library()
    return m


def _rows(V, shift, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.zeros(N, -(-V // 8) * 8, dtype=torch.bfloat16, device=DEV)[:, :V]
    for r in range(0, N, 256):
        x[r:r + 256] = (torch.randn(256, V, generator=g, device=DEV) * 1.5 + shift).bfloat16()
    return x


def _ratio(difr, a, b, T, top_p=0.9):
    """Time of rows `a` over that of rows `b`: the least of several runs each, in turn."""
    row = torch.arange(N, dtype=torch.int32, device=DEV)
    at = (T, torch.tensor([5], device=DEV), row * 0, row, row)
    best = [float("inf")] * 2
    for _ in range(6):
        for k, x in enumerate((a, b)):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(4):
                difr.ipt_score_filtered(x, *at, top_k=0, top_p=top_p)
            t1.record()
            t1.synchronize()
            best[k] = min(best[k], t0.elapsed_time(t1))
    print("time ratio %.2f" % (best[0] / best[1]), flush=True)
    return best[0] / best[1]


# (rows that are counted and then searched take 6 times as long as counted ones here: a bound of 1.4 separates the two)
@pytest.mark.parametrize("shift,T", [(-45.0, 1.2), (0.0, 1.6), (0.0, 0.7)])
def test_a_ragged_end_does_not_send_rows_to_the_search(difr, shift, T):
    print("nucleus routes, ragged", shift, T, flush=True)
    assert _ratio(difr, _rows(50257, shift, 1), _rows(50256, shift, 1), T) < 1.4


@pytest.mark.parametrize("T", [0.7, 1.6])
def test_a_mask_does_not_send_rows_to_the_search(difr, T):
    """(At high temperatures the row is read once more, to see that its low entries are all masked: 1.3 times as long.)"""
    x = _rows(50256, 0.0, 2)
    m = x.clone()
    m[:, 5::20] = -float("inf")
    print("nucleus routes, masked", T, flush=True)
    assert _ratio(difr, m, x, T) < 2.5


# (counted, these rows take 2.7, 2.9 and 5.7 times as long as constant ones, which are searched; searched 1.0, 1.8 and 2.9 times)
@pytest.mark.parametrize("kind,bound", [("two in turn", 1.7), ("period 8", 2.3), ("around zero", 4.0)])
def test_rows_whose_waves_would_queue_at_a_counter_are_searched(difr, kind, bound):
    """Entries that a wave counts at once - eight apart in the row - and that share a counter: a constant row shows it in any pair, these
    in the same place of neighbouring vectors, or on the counter of the values around zero, only."""
    V = 50256
    x = _rows(V, 0.0, 3)
    m = x.clone()
    if kind == "two in turn":
        m[:, ::2], m[:, 1::2] = 1.5, 0.5
    elif kind == "period 8":
        m = x[:, :8].repeat(1, V // 8).contiguous()
    else:
        m[:, torch.rand(V, device=DEV) < 0.9] *= 1e-5
    const = torch.full_like(x, 1.5)
    print("nucleus routes, queues", kind, flush=True)
    assert _ratio(difr, m, const, 0.7) < bound


def test_a_cut_at_zero_does_not_send_rows_of_few_values_to_the_search(difr):
    """Rows of multiples of 1/2 around zero, the cut at zero, against the same rows a step of 1 higher."""
    x = (_rows(50256, 0.0, 4).float() * 2).round() / 2
    print("nucleus routes, cut at zero", flush=True)
    assert _ratio(difr, x.bfloat16(), (x + 1).bfloat16(), 1.0, 0.933) < 1.4
