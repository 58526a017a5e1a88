"""What the nucleus kernel's look at a bf16 row decides, in plain torch: whether the row is counted first or searched at once."""
import math

import torch


def looked_at(V):
    """Positions of the entries looked at: 32 runs of eight vectors, or the whole of a shorter row."""
    nvec = -(-V // 8)
    vec = torch.arange(256)
    if nvec >= 256:
        vec = (vec // 8) * (nvec // 32) + vec % 8
    return vec


def counted_first(x, V, T):
    """For each row of x (bf16, on the CPU): whether its entries are counted before anything else."""
    nvec = -(-V // 8)
    padded = torch.full((x.shape[0], max(nvec, 256) * 8), -math.inf, dtype=torch.bfloat16)
    padded[:, :V] = x[:, :V]
    q = padded.view(x.shape[0], -1, 8)[:, looked_at(V)]                   # [row, thread, place]
    f = q.float()
    R = f.amax((1, 2))
    lo = torch.where(f == -math.inf, math.inf, f).amin((1, 2))
    unusable = ~(R.isfinite())
    if bool(unusable.any()):                                              # a whole pass then finds them
        whole = x[:, :V].float()
        R = torch.where(unusable, whole.amax(1), R)
        lo = torch.where(unusable, torch.where(whole == -math.inf, math.inf, whole).amin(1), lo)
    bits = q.view(torch.int16).int() & 0xFFFF
    m = (bits & 0x7FFF).clamp(min=0x3A80) - 0x3A80
    word = 2239 + torch.where(bits >= 0x8000, -m.clamp(max=2239), m.clamp(max=2239))
    word = torch.where(word < 64, -1 - torch.arange(256).view(1, 256, 1), word)  # (a thread's own)
    word = word[:, :, [0, 1, 4, 5]]
    lane = torch.arange(256)
    equal = sum((word == word[:, lane ^ d]).float().mean((1, 2)) for d in (1, 4)) / 2
    few = torch.ones_like(R, dtype=torch.bool) if nvec < 256 else equal <= min(0.12 + 4500.0 / V, 0.6)
    far = (-127.5 - R) * (1.4426950408889634 / T) < -126.0
    return (R < 128) & ((lo > -128) | far) & few
