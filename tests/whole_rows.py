"""The calls that give every row one workgroup, through their C entry points: the Python functions share the rows of small batches
among workgroups, so a test of that needs these beside them."""
import ctypes as C

import torch

from paper_2511_02620_amd import binding as B


def _p(t):
    return None if t is None else C.c_void_p(t.data_ptr())


def _sides(N, dev, rank=False, token=False, mass=False):
    f, i32, u8 = ((lambda dt: (lambda: torch.empty(N, dtype=dt, device=dev)))(dt) for dt in (torch.float32, torch.int32, torch.uint8))
    g = dict(margin=f(), argmax=i32(), max_score=f(), claimed_score=f(), flags=u8())
    i = dict(dist=f(), cdf_lo=f(), cdf_hi=f(), u=f(), flags=u8())
    if rank:
        g["logit_rank"] = i32()
    if token:
        i["ipt_token"] = i32()
    if mass:
        i["log_mass"] = f()
    return g, i


_G = ("margin", "argmax", "max_score", "claimed_score", "flags")
_I = ("dist", "cdf_lo", "cdf_hi", "u")


def score_both(logits, T, seeds, sid, pos, cg, ci, temperatures=None, V=None, want_rank=False, want_token=False, want_log_mass=False,
               peaked=False):
    lib = B.load_library()
    r, N, dev = B._rows(logits, V, T, seeds, sid, pos, cg, temperatures)
    g, i = _sides(N, dev, want_rank, want_token, want_log_mass)
    rc = (lib.difr_score_both_peaked if peaked else lib.difr_score_both)(
        C.byref(r), _p(ci), *[_p(g[k]) for k in _G], _p(g.get("logit_rank")), *[_p(i[k]) for k in _I], _p(i.get("ipt_token")), 0.01,
        1e-30, _p(i.get("log_mass")), _p(i["flags"]), B._stream_ptr(dev))
    assert rc == 0, rc
    return g, i


def gumbel_score(logits, T, seeds, sid, pos, claims, temperatures=None, V=None, want_rank=False):
    lib = B.load_library()
    r, N, dev = B._rows(logits, V, T, seeds, sid, pos, claims, temperatures)
    g = _sides(N, dev, want_rank)[0]
    rc = lib.difr_gumbel_score(C.byref(r), *[_p(g[k]) for k in _G], _p(g.get("logit_rank")), B._stream_ptr(dev))
    assert rc == 0, rc
    return g


def ipt_score(logits, T, seeds, sid, pos, claims, temperatures=None, V=None):
    lib = B.load_library()
    r, N, dev = B._rows(logits, V, T, seeds, sid, pos, claims, temperatures)
    i = _sides(N, dev)[1]
    rc = lib.difr_ipt_score(C.byref(r), *[_p(i[k]) for k in _I], None, 0.01, 1e-30, None, _p(i["flags"]), None, B._stream_ptr(dev))
    assert rc == 0, rc
    return i


def score_both_admissible(logits, T, seeds, sid, pos, delta, cg, ci, temperatures=None, V=None):
    lib = B.load_library()
    r, N, dev = B._rows(logits, V, T, seeds, sid, pos, cg, temperatures)
    g, i = _sides(N, dev)
    a = dict(count=torch.empty(N, dtype=torch.int32, device=dev), log2_count=torch.empty(N, dtype=torch.float32, device=dev))
    rc = lib.difr_score_both_admissible(C.byref(r), _p(ci), delta, *[_p(g[k]) for k in _G], *[_p(i[k]) for k in _I], _p(i["flags"]),
                                        _p(a["count"]), _p(a["log2_count"]), B._stream_ptr(dev))
    assert rc == 0, rc
    return g, i, a


def is_shared(logits, V=None):
    """Whether the Python functions share the rows of this batch."""
    V = logits.shape[1] if V is None else V
    return B.load_library().difr_split_workspace_bytes(logits.shape[0], V, 0 if logits.dtype == torch.bfloat16 else 1, 0) > 0
