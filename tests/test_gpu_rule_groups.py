"""The vector-unit second score pass on both sides of its workgroup size (64 positions while
256 would leave CUs idle), with odd lengths, a chunk of memory rows more than LDS holds and
dead slots, against float64. float32 logits of order one and sums of up to 14 x 2 x 70 weights:
1e-5 of the value."""
import pytest

from perf import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,R,D", [(1, 63, 1, 64), (1, 2049, 33, 64), (7, 8191, 16, 64), (8, 8191, 16, 64),
                                     (14, 4700, 70, 64), (2, 1300, 65, 128)])
def test_rule_scores(L, N, R, D):
    import torch
    c = cases._case("score", dict(L=L, Hq=8, Hkv=2, D=D, dtype="f32"), N=N, C=N // 4, R=R, span=9, dead=0.1, pi=2,
                    scorer="rule")
    st = cases.prepare(c, N + R)
    want = cases._exact_scores(c, st, 0, st["M"])
    got = cases.run(st)["scores"].double()
    on = want > -float("inf")
    assert torch.equal(on, got > -float("inf"))
    assert bool(((got[on] - want[on]).abs() <= 1e-5 * want[on]).all())
