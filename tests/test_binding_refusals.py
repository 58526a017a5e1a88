"""The native side of the binding refuses what its Python checks refuse, with their messages, and takes every optional
argument in its place (values against the oracle: test_gpu_parity.py and the tests of each call)."""
import pytest
import torch

import paper_2511_02620_amd as difr


def _args(dev, N=4, V=64):
    return dict(logits=torch.zeros(N, V, device=dev), temperature=1.0, seeds=torch.zeros(1, dtype=torch.int64, device=dev),
                seq_ids=torch.zeros(N, dtype=torch.int32, device=dev), positions=torch.zeros(N, dtype=torch.int32, device=dev))


def test_host_tensors_are_refused():
    a = _args("cpu")
    z = torch.zeros(4)
    for call in (lambda: difr.gumbel_score(**a), lambda: difr.ipt_score(**a), lambda: difr.score_both(**a),
                 lambda: difr.score_both_peaked(**a), lambda: difr.score_both_admissible(delta=1.0, **a),
                 lambda: difr.ipt_score_filtered(**a), lambda: difr.gumbel_likelihood(claimed=None, z=z, **a),
                 lambda: difr.score_both_filtered(claimed_gumbel=None, claimed_ipt=None, z=z, **a),
                 lambda: difr.admissible_count(max_score=z, delta=1.0, **a)):
        with pytest.raises(ValueError, match="logits must be a GPU tensor"):
            call()
    for call in (lambda: difr.seq_reduce(z, None, a["seeds"], 0.0), lambda: difr.classify(z, a["seq_ids"], 0.0, 8, 64)):
        with pytest.raises(ValueError, match="scores must be"):
            call()
    with pytest.raises(ValueError, match="hidden must be"):
        difr.lmhead_score(a["logits"], a["logits"], 1.0, a["seeds"], a["seq_ids"], a["positions"])
    with pytest.raises(ValueError):
        difr.gumbel_score(**dict(a, temperature="warm"))


@pytest.mark.gpu
@pytest.mark.parametrize("change, message", [
    (dict(logits=lambda t: t.half()), "bfloat16 or float32"), (dict(logits=lambda t: t.t()), "unit column stride"),
    (dict(logits=lambda t: t[0]), "2-D"), (dict(seq_ids=lambda t: t.long()), "seq_ids"),
    (dict(positions=lambda t: t[:3]), "positions"), (dict(seeds=lambda t: t.cpu()), "seeds"),
    (dict(claimed_ipt=lambda t: t.repeat(2)[::2]), "claimed_ipt"), (dict(temperatures=lambda t: t.double()), "temperatures"),
    (dict(temperature=lambda t: 0.0), "temperature"), (dict(V=lambda t: 65), "shape"), (dict(sigma=lambda t: 0.0), "argument")])
def test_what_is_refused_on_the_device(change, message):
    dev = "cuda:0"
    a = dict(_args(dev), claimed_ipt=torch.zeros(4, dtype=torch.int32, device=dev),
             temperatures=torch.ones(4, device=dev), V=64, sigma=0.01, want_log_mass=True)
    if "temperature" in change:
        a["temperatures"] = None
    for k, f in change.items():
        a[k] = f(a[k])
    with pytest.raises((ValueError, difr.DifrError), match=message):
        difr.score_both(**a)


@pytest.mark.gpu
def test_outputs_are_the_ones_asked_for():
    a = _args("cuda:0")
    assert list(difr.gumbel_score(want_scores=False, **a)) == ["margin", "argmax", "flags"]
    assert list(difr.ipt_score(want_interval=False, want_token=True, want_log_mass=True, want_rank=True, **a)) == [
        "dist", "flags", "ipt_token", "log_mass", "logit_rank"]
    g, i = difr.score_both(want_rank=True, want_token=True, want_log_mass=True, **a)
    assert list(g) == ["margin", "argmax", "max_score", "claimed_score", "flags", "logit_rank"]
    assert list(i) == ["dist", "cdf_lo", "cdf_hi", "u", "flags", "ipt_token", "log_mass"]
    empty = dict(a, logits=a["logits"][:0], seq_ids=a["seq_ids"][:0], positions=a["positions"][:0])
    assert all(t.shape == (0,) for part in difr.score_both(**empty) for t in part.values())
