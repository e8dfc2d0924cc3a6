"""Softmax sums whose reference has to move: logits that rise, fall or jump along the history,
far beyond the slack within which the first score pass and the prefill attention leave a row's
reference where it is. Against float64, at list and row counts around the tile edges.

A bf16 hi + lo product keeps 2^-17 of its size and the logits reach about 60 (natural log), so
a weight is off by up to 60 * 2^-17 = 4.6e-4 of itself: 1e-3 is allowed. The prefill's logits
are of bf16 inputs (exact products), its outputs are rounded to bf16 (2^-9 of the value)."""
import pytest

from paper_2606_09916_amd import ikv
from perf import cases

pytestmark = pytest.mark.gpu
SHAPE = dict(L=2, Hq=8, Hkv=2, D=128, dtype="bf16")


def _ramp(kind, n, dev):
    import torch
    x = torch.linspace(0.05, 4.0, n, device=dev)
    if kind == "fall":
        x = x.flip(0)
    if kind == "jump":
        x = torch.where(torch.arange(n, device=dev) % 97 == 96, 4.0, 0.05)
    return x


def _scale_keys(st, kind):
    S = st["S0"].long()
    st["k"][:, S] = (st["k"][:, S].float() * _ramp(kind, len(S), S.device)[None, :, None, None]).bfloat16()
    ikv.init_dead_slot(st["pool"])


@pytest.mark.parametrize("kind", ["rise", "fall", "jump"])
@pytest.mark.parametrize("N,R,scorer", [(1100, 17, "rule"), (1127, 64, "rule"), (2081, 65, "rule"),
                                        (20033, 128, "rule"), (1100, 31, "snapkv"), (1121, 128, "snapkv")])
def test_scores(kind, N, R, scorer):
    import torch
    c = cases._case("score", SHAPE, N=N, C=300, R=R, span=11, dead=0.1, pi=3, scorer=scorer)
    st = cases.prepare(c, N + R)
    _scale_keys(st, kind)
    st["M"].mul_(30.0 if scorer == "rule" else 2.5)
    got = cases.run(st)["scores"].double()
    want = cases._exact_scores(c, st, 0, st["M"])
    on = want > -float("inf")
    assert torch.equal(on, got > -float("inf"))
    err = (got[on] - want[on]).abs()
    assert bool((err <= 1e-3 * want[on] + 1e-7 * want[on].max()).all()), float((err / want[on].max()).max())


@pytest.mark.parametrize("kind", ["rise", "fall", "jump"])
@pytest.mark.parametrize("N,span", [(63, 9), (64, 64), (1000, 13), (7001, 33)])
def test_prefill(kind, N, span):
    c = cases._case("prefill", SHAPE, N=N, span=span)
    st = cases.prepare(c, N)
    _scale_keys(st, kind)
    want = cases._exact_prefill(c, st)["out"]
    got = cases.run(st)["out"].double()
    err = (got - want).abs()
    # the split of the weights keeps 2^-17 of values of order one
    assert bool((err <= want.abs() * 2.0 ** -8 + 1e-4).all()), float(err.max())


# Logits that begin far below zero (-300 natural): a row's first reference is set by a downward
# move, from nothing. "deep": the whole history; "climb": the first 32 list entries of every
# 128 positions and more, the rest near zero. The offset is 64 in one channel of the rows
# against -53 in the keys, exact in bf16, so the float32 sums alone count: a few units of 433
# (log2) times 2^-24 each, 1e-4 of a weight.

def _offset(kind, n, dev):
    import torch
    o = torch.full((n,), -53.0, device=dev)
    if kind == "climb":
        o[torch.arange(n, device=dev) % 128 >= 80] = 0.0
    return o


@pytest.mark.parametrize("kind", ["deep", "climb"])
@pytest.mark.parametrize("N,R,scorer", [(1100, 17, "rule"), (1127, 64, "rule"), (2081, 65, "rule"),
                                        (20033, 128, "rule"), (1100, 4, "two_pass"), (1121, 128, "snapkv")])
def test_scores_from_far_below(kind, N, R, scorer):
    import torch
    c = cases._case("score", SHAPE, N=N, C=300, R=R, span=11, dead=0.1, pi=3,
                    scorer="rule" if scorer == "two_pass" else scorer)
    st = cases.prepare(c, N + R)
    S = st["S0"].long()
    st["k"][:, S, :, 0] = _offset(kind, len(S), S.device)[None, :, None].bfloat16()
    ikv.init_dead_slot(st["pool"])
    if scorer != "snapkv":
        st["M"].mul_(4.0)
    st["M"].view(-1, 128)[:, 0] = 64.0
    if scorer == "two_pass":
        ikv.score_history(st["pool"], st["sess"], st["S"], st["M"], st["scores"], st["ws"], flags=ikv.IKV_TWO_PASS)
    else:
        cases.run(st)
    got = st["scores"].double()
    want = cases._exact_scores(c, st, 0, st["M"])
    on = want > -float("inf")
    assert torch.equal(on, got > -float("inf"))
    err = (got[on] - want[on]).abs()
    assert bool((err <= 1e-3 * want[on] + 1e-7 * want[on].max()).all()), float((err / want[on].max()).max())


@pytest.mark.parametrize("kind", ["deep", "climb"])
@pytest.mark.parametrize("N,span", [(63, 9), (1000, 13), (7001, 33)])
def test_prefill_from_far_below(kind, N, span):
    """The offset sits in the channel pair that turns slowest (0.01 rad at 7000 positions)."""
    c = cases._case("prefill", SHAPE, N=N, span=span)
    st = cases.prepare(c, N)
    S = st["S0"][:N].long()
    st["k"][:, S, :, 63] = _offset(kind, N, S.device)[None, :, None].bfloat16()
    ikv.init_dead_slot(st["pool"])
    st["q_raw"].view(-1, 128)[:, 63] = 64.0
    st["k_raw"].view(-1, 128)[:, 63] = -53.0 if kind == "deep" else 0.0
    want = cases._exact_prefill(c, st)["out"]
    got = cases.run(st)["out"].double()
    err = (got - want).abs()
    # values of order four: 1e-4 of a weight on either side of the sum
    assert bool((err <= want.abs() * 2.0 ** -8 + 1e-3).all()), float(err.max())
