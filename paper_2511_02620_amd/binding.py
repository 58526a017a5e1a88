"""Binding of libdifr.so: argument marshalling only.

Every function takes torch tensors that already live on the GPU, hands their device
pointers and the current HIP stream to the C entry point of the same name, and returns
freshly allocated output tensors.  No arithmetic of the method happens here.  The calls of
the hot path are marshalled in native code (csrc/binding.cpp); the audit helpers, the
allocation-free LM-head call and every check's error message are ctypes and Python.
"""
from __future__ import annotations

import ctypes as C
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libdifr.so")
_lib = None
_native = None

FLAG_MATCH = 1
FLAG_INVALID_CLAIM = 2
FLAG_NONFINITE = 4
FLAG_SLOW_PATH = 8

DTYPE_BF16 = 0
DTYPE_F32 = 1


class DifrError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        msg = load_library().difr_status_string(status).decode()
        super().__init__("%s: difr_status %d (%s)" % (where, status, msg))


class _Rows(C.Structure):
    _fields_ = [
        ("logits", C.c_void_p),
        ("dtype", C.c_int32),
        ("N", C.c_int64),
        ("V", C.c_int64),
        ("ld", C.c_int64),
        ("temperature", C.c_float),
        ("temperatures", C.c_void_p),
        ("seeds", C.c_void_p),
        ("S", C.c_int64),
        ("seq_ids", C.c_void_p),
        ("positions", C.c_void_p),
        ("claimed", C.c_void_p),
    ]


class _LmHead(C.Structure):
    _fields_ = [
        ("hidden", C.c_void_p),
        ("weight", C.c_void_p),
        ("N", C.c_int64),
        ("V", C.c_int64),
        ("d", C.c_int64),
        ("ldh", C.c_int64),
        ("ldw", C.c_int64),
        ("temperature", C.c_float),
        ("temperatures", C.c_void_p),
        ("seeds", C.c_void_p),
        ("S", C.c_int64),
        ("seq_ids", C.c_void_p),
        ("positions", C.c_void_p),
        ("claimed_gumbel", C.c_void_p),
        ("claimed_ipt", C.c_void_p),
    ]


class _Scores(C.Structure):
    _fields_ = [("margin", C.c_void_p), ("argmax", C.c_void_p), ("max_score", C.c_void_p), ("claimed_score", C.c_void_p),
                ("flags_gumbel", C.c_void_p), ("rank_gumbel", C.c_void_p), ("dist", C.c_void_p), ("cdf_lo", C.c_void_p),
                ("cdf_hi", C.c_void_p), ("u", C.c_void_p), ("ipt_token", C.c_void_p), ("sigma", C.c_double),
                ("eps", C.c_double), ("log_mass", C.c_void_p), ("flags_ipt", C.c_void_p), ("rank_ipt", C.c_void_p),
                ("delta", C.c_float), ("count", C.c_void_p), ("log2_count", C.c_void_p)]


class _LikelihoodParams(C.Structure):
    _fields_ = [("top_k", C.c_int32), ("top_p", C.c_float), ("s", C.c_int32), ("sigma", C.c_float),
                ("M", C.c_int32), ("z", C.c_void_p)]


EXPORTS = ("difr_gumbel_score", "difr_debug_gumbel_score_unfiltered", "difr_ipt_score", "difr_score_both", "difr_score_both_peaked", "difr_score_both_admissible", "difr_admissible_count", "difr_gumbel_likelihood", "difr_ipt_score_filtered", "difr_score_both_filtered", "difr_lmhead_score", "difr_lmhead_score_static", "difr_lmhead_workspace_bytes", "difr_split_workspace_bytes", "difr_score_split", "difr_classify", "difr_seq_reduce", "difr_debug_noise", "difr_debug_gumbel_map",
           "difr_philox4x32_10", "difr_status_string", "difr_version")


def lib_path() -> str:
    return _LIB_PATH


def load_library():
    """Load libdifr.so.  Raises if it has not been built: there is no fallback path."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError("libdifr.so is missing at %s: build it with `python -m paper_2511_02620_amd.build` "
                          "(there is no CPU fallback)" % _LIB_PATH)
    lib = C.CDLL(_LIB_PATH)
    vp = C.c_void_p
    lib.difr_gumbel_score.argtypes = [C.POINTER(_Rows), vp, vp, vp, vp, vp, vp, vp]
    lib.difr_gumbel_score.restype = C.c_int
    lib.difr_debug_gumbel_score_unfiltered.argtypes = [C.POINTER(_Rows), vp, vp, vp, vp, vp, vp, vp]
    lib.difr_debug_gumbel_score_unfiltered.restype = C.c_int
    lib.difr_ipt_score.argtypes = [C.POINTER(_Rows), vp, vp, vp, vp, vp, C.c_double, C.c_double, vp, vp, vp, vp]
    lib.difr_score_both.argtypes = [C.POINTER(_Rows)] + [vp] * 12 + [C.c_double, C.c_double, vp, vp, vp]
    lib.difr_score_both.restype = C.c_int
    lib.difr_score_both_peaked.argtypes = lib.difr_score_both.argtypes
    lib.difr_score_both_peaked.restype = C.c_int
    lib.difr_score_both_admissible.argtypes = [C.POINTER(_Rows), vp, C.c_float] + [vp] * 13
    lib.difr_score_both_admissible.restype = C.c_int
    lib.difr_ipt_score_filtered.argtypes = [C.POINTER(_Rows), C.c_int32, C.c_float, vp, vp, vp, vp, vp, C.c_double,
                                            C.c_double, vp, vp, vp, vp]
    lib.difr_ipt_score_filtered.restype = C.c_int
    lib.difr_gumbel_likelihood.argtypes = [C.POINTER(_Rows), C.POINTER(_LikelihoodParams), vp, vp, vp, vp, vp, vp]
    lib.difr_gumbel_likelihood.restype = C.c_int
    lib.difr_score_both_filtered.argtypes = [C.POINTER(_Rows), vp, C.POINTER(_LikelihoodParams)] + [vp] * 10 + [
        C.c_double, C.c_double, vp, vp, vp, vp]
    lib.difr_score_both_filtered.restype = C.c_int
    lib.difr_admissible_count.argtypes = [C.POINTER(_Rows), vp, C.c_float, vp, vp, vp]
    lib.difr_admissible_count.restype = C.c_int
    lib.difr_lmhead_workspace_bytes.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_int32]
    lib.difr_lmhead_workspace_bytes.restype = C.c_size_t
    lib.difr_lmhead_score.argtypes = [C.POINTER(_LmHead)] + [vp] * 11 + [C.c_double, C.c_double, vp, vp, vp, C.c_size_t, vp]
    lib.difr_lmhead_score.restype = C.c_int
    lib.difr_lmhead_score_static.argtypes = [C.POINTER(_LmHead)] + [vp] * 10 + [C.c_double, C.c_double, vp, vp, vp]
    lib.difr_lmhead_score_static.restype = C.c_int
    lib.difr_split_workspace_bytes.argtypes = [C.c_int64, C.c_int64, C.c_int32, C.c_int32]
    lib.difr_split_workspace_bytes.restype = C.c_size_t
    lib.difr_score_split.argtypes = [C.POINTER(_Rows), vp, C.POINTER(_Scores), vp, C.c_size_t, vp]
    lib.difr_score_split.restype = C.c_int
    lib.difr_classify.argtypes = [vp, vp, C.c_int64, C.c_float, C.c_int64, C.c_int64, vp, vp, vp, vp]
    lib.difr_classify.restype = C.c_int
    lib.difr_ipt_score.restype = C.c_int
    lib.difr_seq_reduce.argtypes = [vp, vp, vp, C.c_int64, C.c_int64, C.c_float, vp, vp, vp, vp, vp]
    lib.difr_seq_reduce.restype = C.c_int
    lib.difr_debug_noise.argtypes = [C.POINTER(_Rows), C.c_int64, C.c_int32, vp, vp]
    lib.difr_debug_noise.restype = C.c_int
    lib.difr_debug_gumbel_map.argtypes = [vp, C.c_int64, vp, vp]
    lib.difr_debug_gumbel_map.restype = C.c_int
    lib.difr_philox4x32_10.argtypes = [C.POINTER(C.c_uint32), C.POINTER(C.c_uint32), C.POINTER(C.c_uint32)]
    lib.difr_philox4x32_10.restype = None
    lib.difr_status_string.argtypes = [C.c_int]
    lib.difr_status_string.restype = C.c_char_p
    lib.difr_version.argtypes = []
    lib.difr_version.restype = C.c_int
    _lib = lib
    return lib


def _load_native():
    """The native side of this binding (csrc/binding.cpp), with the addresses of the library's entry points."""
    global _native
    lib = load_library()
    try:
        from . import _native as native
    except ImportError as e:
        raise ImportError("_native.so is missing or does not load: build it with `python -m paper_2511_02620_amd.build`") from e
    native.bind({name: C.cast(getattr(lib, name), C.c_void_p).value for name in EXPORTS})
    _native = native
    return native


def version() -> int:
    return int(load_library().difr_version())


def philox4x32_10(ctr, key):
    """Host helper: one Philox4x32-10 block (4 counter words, 2 key words) -> 4 words."""
    c = (C.c_uint32 * 4)(*[int(x) & 0xFFFFFFFF for x in ctr])
    k = (C.c_uint32 * 2)(*[int(x) & 0xFFFFFFFF for x in key])
    out = (C.c_uint32 * 4)()
    load_library().difr_philox4x32_10(c, k, out)
    return [int(x) for x in out]


def _stream_ptr(device) -> int:
    return int(torch.cuda.current_stream(device).cuda_stream)


def _ptr(t):
    return None if t is None else C.c_void_p(t.data_ptr())


def _check(t, dtype, n, name, device):
    if t is None:
        return
    if t.device != device:
        raise ValueError("%s must live on %s" % (name, device))
    if t.dtype != dtype or t.dim() != 1 or t.shape[0] != n or not t.is_contiguous():
        raise ValueError("%s must be a contiguous 1-D %s tensor of %d elements" % (name, dtype, n))


def _rows(logits, V, temperature, seeds, seq_ids, positions, claimed, temperatures):
    if not logits.is_cuda:
        raise ValueError("logits must be a GPU tensor")
    if logits.dim() != 2 or logits.stride(1) != 1 and logits.shape[1] > 1:
        raise ValueError("logits must be 2-D with unit column stride")
    if logits.dtype == torch.bfloat16:
        dt = DTYPE_BF16
    elif logits.dtype == torch.float32:
        dt = DTYPE_F32
    else:
        raise ValueError("logits must be bfloat16 or float32")
    dev = logits.device
    N = logits.shape[0]
    V = logits.shape[1] if V is None else int(V)
    ld = logits.stride(0) if N > 1 else max(logits.shape[1], logits.stride(0) if N else 0)
    _check(seq_ids, torch.int32, N, "seq_ids", dev)
    _check(positions, torch.int32, N, "positions", dev)   # uint32 bit patterns held in int32
    _check(claimed, torch.int32, N, "claimed", dev)
    _check(temperatures, torch.float32, N, "temperatures", dev)
    if seeds.device != dev or seeds.dtype != torch.int64 or seeds.dim() != 1 or not seeds.is_contiguous():
        raise ValueError("seeds must be a contiguous 1-D int64 GPU tensor (uint64 bit patterns)")
    r = _Rows()
    r.logits = logits.data_ptr()
    r.dtype = dt
    r.N, r.V, r.ld = N, V, ld
    r.temperature = float(temperature)
    r.temperatures = None if temperatures is None else temperatures.data_ptr()
    r.seeds = seeds.data_ptr()
    r.S = seeds.shape[0]
    r.seq_ids = seq_ids.data_ptr()
    r.positions = positions.data_ptr()
    r.claimed = None if claimed is None else claimed.data_ptr()
    return r, N, dev


def _refused(name, rc, checks):
    """The native call handed back no tensors: raise what is wrong (rc: the difr_status of the entry point, or None if an
    argument is not what it has to be, which `checks` then names)."""
    if rc is None:
        checks()
        raise ValueError("%s: an argument is not a tensor of the kind the call takes" % name)
    raise DifrError(rc, name)


def _check_z(z, dev):
    if z.device != dev or z.dtype != torch.float32 or z.dim() != 1 or not z.is_contiguous():
        raise ValueError("z must be a contiguous 1-D float32 tensor on the device of logits")


def gumbel_score(logits, temperature, seeds, seq_ids, positions, claimed=None, temperatures=None, V=None,
                 want_scores=True, unfiltered=False, want_rank=False):
    """difr_gumbel_score (or, with unfiltered=True, difr_debug_gumbel_score_unfiltered).
    logits [N, >=V] bf16/fp32 on the GPU; seeds int64 [S] (uint64 bits); seq_ids, positions,
    claimed int32 [N].  Returns a dict of device tensors."""
    out = (_native or _load_native()).gumbel_score(logits, V if V is None else int(V), float(temperature), seeds, seq_ids, positions,
                                                   claimed, temperatures, want_scores, unfiltered, want_rank)
    if out.__class__ is not dict:
        _refused("difr_gumbel_score", out,
                 lambda: _rows(logits, V, temperature, seeds, seq_ids, positions, claimed, temperatures))
    return out


def ipt_score(logits, temperature, seeds, seq_ids, positions, claimed=None, temperatures=None, V=None,
              want_token=False, want_log_mass=False, sigma=0.01, eps=1e-30, want_interval=True, want_rank=False):
    """difr_ipt_score.  Same inputs as :func:`gumbel_score`.  Returns a dict of device tensors.

    The rows of a small batch of long rows are shared among workgroups (difr_score_split), which add up a row's softmax sum in
    another order: dist, cdf_lo, cdf_hi and log_mass of the same row may differ in their last bits between batches of different
    size, and MATCH and ipt_token where u lies that near to an interval's edge.  The C entry point adds in one order always."""
    out = (_native or _load_native()).ipt_score(logits, V if V is None else int(V), float(temperature), seeds, seq_ids, positions,
                                                claimed, temperatures, want_token, want_log_mass, float(sigma), float(eps),
                                                want_interval, want_rank)
    if out.__class__ is not dict:
        _refused("difr_ipt_score", out,
                 lambda: _rows(logits, V, temperature, seeds, seq_ids, positions, claimed, temperatures))
    return out


def score_both(logits, temperature, seeds, seq_ids, positions, claimed_gumbel=None, claimed_ipt=None,
               temperatures=None, V=None, want_rank=False, want_token=False, want_log_mass=False, sigma=0.01, eps=1e-30):
    """difr_score_both: both estimators in one pass.  Returns (gumbel dict, ipt dict) of device tensors;
    want_rank adds logit_rank (of the Token-DiFR claim) to the first, want_token / want_log_mass add ipt_token /
    log_mass to the second (as in :func:`ipt_score`, which
    also says what depends on the size of the batch: nothing of the first dict, the last bits of the second)."""
    return _score_both("difr_score_both", False, logits, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt,
                       temperatures, V, want_rank, want_token, want_log_mass, sigma, eps)


def score_both_peaked(logits, temperature, seeds, seq_ids, positions, claimed_gumbel=None, claimed_ipt=None,
                      temperatures=None, V=None, want_rank=False, want_token=False, want_log_mass=False, sigma=0.01,
                      eps=1e-30):
    """difr_score_both_peaked: :func:`score_both` for rows known to be concentrated; same arguments, same results (to the last
    bits of the second dict: up to 320 rows of a small batch are shared among workgroups, as :func:`score_both` shares them)."""
    return _score_both("difr_score_both_peaked", True, logits, temperature, seeds, seq_ids, positions, claimed_gumbel,
                       claimed_ipt, temperatures, V, want_rank, want_token, want_log_mass, sigma, eps)


def _check_pair(logits, V, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt, temperatures):
    r, N, dev = _rows(logits, V, temperature, seeds, seq_ids, positions, claimed_gumbel, temperatures)
    _check(claimed_ipt, torch.int32, N, "claimed_ipt", dev)
    return dev


def _score_both(entry_name, peaked, logits, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt, temperatures, V,
                want_rank, want_token, want_log_mass, sigma, eps):
    out = (_native or _load_native()).score_both(logits, V if V is None else int(V), float(temperature), seeds, seq_ids, positions,
                                                 claimed_gumbel, temperatures, claimed_ipt, peaked, want_rank, want_token,
                                                 want_log_mass, float(sigma), float(eps))
    if out.__class__ is not tuple:
        _refused(entry_name, out, lambda: _check_pair(logits, V, temperature, seeds, seq_ids, positions, claimed_gumbel,
                                                      claimed_ipt, temperatures))
    return out


def score_both_admissible(logits, temperature, seeds, seq_ids, positions, delta, claimed_gumbel=None, claimed_ipt=None,
                          temperatures=None, V=None):
    """difr_score_both_admissible: both estimators and the admissible-set size in one pass.
    Returns (gumbel dict, ipt dict, admissible dict with count [-1 = undetermined] and log2_count).  Small batches as in
    :func:`ipt_score`; their counts are always determined."""
    out = (_native or _load_native()).score_both_admissible(logits, V if V is None else int(V), float(temperature), seeds, seq_ids,
                                                            positions, claimed_gumbel, temperatures, claimed_ipt, float(delta))
    if out.__class__ is not tuple:
        _refused("difr_score_both_admissible", out, lambda: _check_pair(logits, V, temperature, seeds, seq_ids, positions,
                                                                        claimed_gumbel, claimed_ipt, temperatures))
    return out


def ipt_score_filtered(logits, temperature, seeds, seq_ids, positions, claimed=None, top_k=50, top_p=1.0,
                       temperatures=None, V=None, want_token=False, want_log_mass=False, sigma=0.01, eps=1e-30):
    """difr_ipt_score_filtered.  Returns a dict of device tensors (dist, cdf_lo, cdf_hi, u, kept, flags, ...)."""
    out = (_native or _load_native()).ipt_score_filtered(logits, V if V is None else int(V), float(temperature), seeds, seq_ids,
                                                         positions, claimed, temperatures, int(top_k), float(top_p), want_token,
                                                         want_log_mass, float(sigma), float(eps))
    if out.__class__ is not dict:
        _refused("difr_ipt_score_filtered", out,
                 lambda: _rows(logits, V, temperature, seeds, seq_ids, positions, claimed, temperatures))
    return out


def gumbel_likelihood(logits, temperature, seeds, seq_ids, positions, claimed, z, top_k=0, top_p=1.0, s=16, sigma=1.0,
                      temperatures=None, V=None, want_active=False):
    """difr_gumbel_likelihood.  z: fp32 [M] standard normal draws on the GPU.  Returns a dict of device tensors."""
    out = (_native or _load_native()).gumbel_likelihood(logits, V if V is None else int(V), float(temperature), seeds, seq_ids,
                                                        positions, claimed, temperatures, z, int(top_k), float(top_p), int(s),
                                                        float(sigma), want_active)
    if out.__class__ is not dict:
        _refused("difr_gumbel_likelihood", out,
                 lambda: _check_z(z, _rows(logits, V, temperature, seeds, seq_ids, positions, claimed, temperatures)[2]))
    return out


def score_both_filtered(logits, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt, z, top_k=50,
                        top_p=1.0, s=16, sigma=1.0, temperatures=None, V=None, want_active=False, want_token=False,
                        want_log_mass=False, sigma_ipt=0.01, eps=1e-30):
    """difr_score_both_filtered: gumbel_likelihood and ipt_score_filtered in one pass over the logits.
    Returns (likelihood dict, filtered-IPT dict), each as the single call returns it."""
    out = (_native or _load_native()).score_both_filtered(logits, V if V is None else int(V), float(temperature), seeds, seq_ids,
                                                          positions, claimed_gumbel, temperatures, z, int(top_k), float(top_p),
                                                          int(s), float(sigma), want_active, claimed_ipt, want_token,
                                                          want_log_mass, float(sigma_ipt), float(eps))
    if out.__class__ is not tuple:
        _refused("difr_score_both_filtered", out,
                 lambda: _check_z(z, _check_pair(logits, V, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt,
                                                 temperatures)))
    return out


def admissible_count(logits, temperature, seeds, seq_ids, positions, max_score, delta, temperatures=None, V=None,
                     want_log2=True):
    """difr_admissible_count: size of { v : max_score - y_v <= delta } per row (max_score from gumbel_score)."""
    out = (_native or _load_native()).admissible_count(logits, V if V is None else int(V), float(temperature), seeds, seq_ids,
                                                       positions, None, temperatures, max_score, float(delta), want_log2)
    if out.__class__ is not dict:
        def checks():
            r, N, dev = _rows(logits, V, temperature, seeds, seq_ids, positions, None, temperatures)
            _check(max_score, torch.float32, N, "max_score", dev)
        _refused("difr_admissible_count", out, checks)
    return out


def lmhead_workspace_bytes(N, V, d, want_token=False) -> int:
    """Bytes of workspace for :func:`lmhead_score`; the size for a batch of up to 256 tokens serves every smaller one."""
    return int(load_library().difr_lmhead_workspace_bytes(int(N), int(V), int(d), int(bool(want_token))))


def _lmhead_args(hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt, temperatures):
    for name, t in (("hidden", hidden), ("weight", weight)):
        if not t.is_cuda or t.dtype != torch.bfloat16 or t.dim() != 2 or (t.shape[1] > 1 and t.stride(1) != 1):
            raise ValueError("%s must be a 2-D bfloat16 GPU tensor with unit column stride" % name)
    dev = hidden.device
    N, d = hidden.shape
    V = weight.shape[0]
    if weight.shape[1] != d or weight.device != dev:
        raise ValueError("weight must be [V, d] on the device of hidden")
    _check(seq_ids, torch.int32, N, "seq_ids", dev)
    _check(positions, torch.int32, N, "positions", dev)
    _check(claimed_gumbel, torch.int32, N, "claimed_gumbel", dev)
    _check(claimed_ipt, torch.int32, N, "claimed_ipt", dev)
    _check(temperatures, torch.float32, N, "temperatures", dev)
    if seeds.device != dev or seeds.dtype != torch.int64 or seeds.dim() != 1 or not seeds.is_contiguous():
        raise ValueError("seeds must be a contiguous 1-D int64 GPU tensor (uint64 bit patterns)")
    r = _LmHead()
    r.hidden, r.weight = hidden.data_ptr(), weight.data_ptr()
    r.N, r.V, r.d = N, V, d
    r.ldh = hidden.stride(0) if N > 1 else d
    r.ldw = weight.stride(0) if V > 1 else d
    r.temperature = float(temperature)
    r.temperatures = None if temperatures is None else temperatures.data_ptr()
    r.seeds, r.S = seeds.data_ptr(), seeds.shape[0]
    r.seq_ids, r.positions = seq_ids.data_ptr(), positions.data_ptr()
    r.claimed_gumbel = None if claimed_gumbel is None else claimed_gumbel.data_ptr()
    r.claimed_ipt = None if claimed_ipt is None else claimed_ipt.data_ptr()
    return r, dev, N, V, d


_LMHEAD_OUT = (("margin", torch.float32), ("argmax", torch.int32), ("max_score", torch.float32),
               ("claimed_score", torch.float32), ("flags", torch.uint8)), (
    ("dist", torch.float32), ("cdf_lo", torch.float32), ("cdf_hi", torch.float32), ("u", torch.float32),
    ("flags", torch.uint8))
_LMHEAD_OPT = (("logit_rank", torch.int32),), (("log_mass", torch.float32), ("ipt_token", torch.int32))


def lmhead_outputs(N, device, want_rank=False, want_log_mass=False, want_token=False):
    """Output buffers of lmhead_score / lmhead_score_static, allocated once and reusable across calls."""
    g, i = tuple({k: torch.empty(N, dtype=dt, device=device) for k, dt in part} for part in _LMHEAD_OUT)
    if want_rank:
        g["logit_rank"] = torch.empty(N, dtype=torch.int32, device=device)
    if want_log_mass:
        i["log_mass"] = torch.empty(N, dtype=torch.float32, device=device)
    if want_token:
        i["ipt_token"] = torch.empty(N, dtype=torch.int32, device=device)
    return g, i


def _lmhead_out(out, N, dev, want_rank, want_log_mass, want_token=False):
    if out is None:
        return lmhead_outputs(N, dev, want_rank, want_log_mass, want_token)
    g, i = out
    for part, spec, opt in zip((g, i), _LMHEAD_OUT, _LMHEAD_OPT):
        for k, dt in spec:
            _check(part[k], dt, N, k, dev)
        for k, dt in opt:
            _check(part.get(k), dt, N, k, dev)
    return g, i


def _lmhead_call(entry_name, token, tail, r, g, i, sigma, eps, dev):
    lib = load_library()
    with torch.cuda.device(dev):
        rc = getattr(lib, entry_name)(C.byref(r), _ptr(g["margin"]), _ptr(g["argmax"]), _ptr(g["max_score"]),
                                      _ptr(g["claimed_score"]), _ptr(g["flags"]), _ptr(g.get("logit_rank")),
                                      _ptr(i["dist"]), _ptr(i["cdf_lo"]), _ptr(i["cdf_hi"]), _ptr(i["u"]), *token,
                                      float(sigma), float(eps), _ptr(i.get("log_mass")), _ptr(i["flags"]), *tail,
                                      _stream_ptr(dev))
    if rc:
        raise DifrError(rc, entry_name)
    return g, i


def lmhead_score(hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel=None, claimed_ipt=None,
                 temperatures=None, workspace=None, out=None, want_rank=False, want_log_mass=False, want_token=False,
                 sigma=0.01, eps=1e-30):
    """difr_lmhead_score: both estimators on logits = hidden @ weight.T that are never stored.
    hidden [N, d], weight [V, d] bf16 on the GPU (unit column stride).  Returns (gumbel dict, ipt dict);
    want_rank adds logit_rank (of the Token-DiFR claim) to the first, want_log_mass / want_token add log_mass /
    ipt_token (the sampler's own token; it needs a larger workspace: lmhead_workspace_bytes(..., want_token=True)) to the second;
    `out` = a pair from lmhead_outputs() to write into instead of new tensors (it decides which optional outputs
    are produced)."""
    if out is None:
        got = (_native or _load_native()).lmhead_score(hidden, weight, float(temperature), seeds, seq_ids, positions, claimed_gumbel,
                                                       claimed_ipt, temperatures, workspace, want_rank, want_log_mass, want_token,
                                                       float(sigma), float(eps))
        if got.__class__ is tuple:
            return got
        if got is not None:
            raise DifrError(got, "difr_lmhead_score")
    r, dev, N, V, d = _lmhead_args(hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt,
                                   temperatures)
    g, i = _lmhead_out(out, N, dev, want_rank, want_log_mass, want_token)
    need = lmhead_workspace_bytes(N, V, d, "ipt_token" in i)
    if workspace is None:
        workspace = torch.empty(max(need, 8), dtype=torch.uint8, device=dev)
    elif workspace.device != dev or workspace.dtype != torch.uint8 or not workspace.is_contiguous():
        raise ValueError("workspace must be a contiguous uint8 tensor on the device of hidden")
    return _lmhead_call("difr_lmhead_score", (_ptr(i.get("ipt_token")),), (_ptr(workspace), workspace.numel()), r, g, i,
                        sigma, eps, dev)


LMHEAD_STATIC_SCRATCH_BYTES = 4 << 20


def lmhead_score_static(hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel=None, claimed_ipt=None,
                        temperatures=None, out=None, want_rank=False, want_log_mass=False, sigma=0.01, eps=1e-30):
    """difr_lmhead_score_static: lmhead_score without a workspace (the library's built-in buffer serves; calls that
    overlap in time on one GPU race on it).  With `out` given (lmhead_outputs()) nothing is allocated at all."""
    r, dev, N, V, d = _lmhead_args(hidden, weight, temperature, seeds, seq_ids, positions, claimed_gumbel, claimed_ipt,
                                   temperatures)
    g, i = _lmhead_out(out, N, dev, want_rank, want_log_mass)
    if "ipt_token" in i:
        raise ValueError("difr_lmhead_score_static has no ipt_token output")
    return _lmhead_call("difr_lmhead_score_static", (), (), r, g, i, sigma, eps, dev)


def seq_reduce(scores, row_flags, seq_offsets, threshold):
    """difr_seq_reduce.  scores fp32 [N], row_flags uint8 [N] or None, seq_offsets int64 [S+1]."""
    out = (_native or _load_native()).seq_reduce(scores, row_flags, seq_offsets, float(threshold))
    if out.__class__ is not dict:
        def checks():
            dev = _check_scores(scores)
            _check(row_flags, torch.uint8, scores.shape[0], "row_flags", dev)
            raise ValueError("seq_offsets must be a contiguous 1-D int64 GPU tensor of S+1 elements")
        _refused("difr_seq_reduce", out, checks)
    return out


def _check_scores(scores):
    if not scores.is_cuda or scores.dtype != torch.float32 or scores.dim() != 1 or not scores.is_contiguous():
        raise ValueError("scores must be a contiguous 1-D float32 GPU tensor")
    return scores.device


def classify(scores, ranks, tau, rank_cutoff, V, log2_admissible=None):
    """difr_classify.  scores fp32 [N], ranks int32 [N] on the GPU.  Returns dict(cls uint8, bits fp32)."""
    out = (_native or _load_native()).classify(scores, ranks, float(tau), int(rank_cutoff), int(V), log2_admissible)
    if out.__class__ is not dict:
        def checks():
            dev, N = _check_scores(scores), scores.shape[0]
            _check(ranks, torch.int32, N, "ranks", dev)
            _check(log2_admissible, torch.float32, N, "log2_admissible", dev)
        _refused("difr_classify", out, checks)
    return out


def debug_noise(logits, temperature, seeds, seq_ids, positions, row, stream, V=None):
    """difr_debug_noise: raw noise words (int32 tensor holding uint32 bits) of one row."""
    lib = load_library()
    r, N, dev = _rows(logits, V, temperature, seeds, seq_ids, positions, None, None)
    bits = torch.empty(int(r.V), dtype=torch.int32, device=dev)
    with torch.cuda.device(dev):
        rc = lib.difr_debug_noise(C.byref(r), int(row), int(stream), _ptr(bits), _stream_ptr(dev))
    if rc:
        raise DifrError(rc, "difr_debug_noise")
    return bits


def debug_gumbel_map(bits):
    """difr_debug_gumbel_map: device bits -> Gumbel map for an int32 tensor of raw words."""
    lib = load_library()
    if not bits.is_cuda or bits.dtype != torch.int32 or not bits.is_contiguous():
        raise ValueError("bits must be a contiguous int32 GPU tensor")
    g = torch.empty(bits.numel(), dtype=torch.float32, device=bits.device)
    with torch.cuda.device(bits.device):
        rc = lib.difr_debug_gumbel_map(_ptr(bits), bits.numel(), _ptr(g), _stream_ptr(bits.device))
    if rc:
        raise DifrError(rc, "difr_debug_gumbel_map")
    return g
