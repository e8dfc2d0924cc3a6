"""The position-major score passes in narrow tiles (k_score_narrow): calls whose candidates
fill at most 512 groups of 32 list entries. Against the float64 oracle at the edges of the
groups, of the key stages (units in fours and twos) and of the memory-row slices; and bit
for bit against the 128-entry passes, which the same session takes beside a long one in a
batch (with one or two units the lists' chunks are 128 positions in both calls, so that
every sum has the same order)."""
import numpy as np
import pytest

import oracle
import synth
from paper_2606_09916_amd import ikv
from paper_2606_09916_amd.step import RetentionStep
from parity import RESID_MFMA_FLOOR, SCORE_FLOOR, check_scores

pytestmark = pytest.mark.gpu


def _session(N, R, dead=0.0):
    return synth.SessionSpec(N=N, C=max(8, N // 4), pi=min(8, N // 8), qs=N - min(24, N // 4), qe=N, R=R, dead_frac=dead)


def _launched(f):
    """Names of the kernels that f() launches."""
    ikv.timing(True)
    try:
        f()
        return [n for n, _ in ikv.timing_read()]
    finally:
        ikv.timing(False)


def _narrow(names):
    """Whether the narrow passes ran; the 128-entry ones then did not, and the other way round."""
    narrow = any(n.startswith("k_score_narrow") for n in names)
    assert narrow != any(n == "k_score_once" or n.startswith("k_score_ws") for n in names), names
    return narrow


def _scores(dev, batch, blob, flags, narrow):
    st = RetentionStep(batch, dev, residual=blob, flags=flags)
    st.init_dead_slot()
    assert _narrow(_launched(st.score)) == narrow
    return st.host("scores")


@pytest.mark.parametrize("flags", [0, ikv.IKV_RESIDUAL])
@pytest.mark.parametrize("N,R,L,Hkv,dead", [
    (40, 5, 3, 1, 0.0), (97, 4, 1, 2, 0.0),         # one and a few groups; a short last stage
    (700, 16, 5, 2, 0.3), (1031, 3, 7, 2, 0.0),
    (8200, 5, 3, 2, 0.0), (16384, 4, 2, 2, 0.1),    # just past 256 groups; the most of one round of pairs
    (16390, 4, 1, 2, 0.0),                          # the 128-entry passes
    (500, 17, 2, 2, 0.0), (3000, 64, 3, 2, 0.2), (9000, 48, 1, 2, 0.0), (2000, 33, 2, 1, 0.0),
    (12000, 16, 2, 2, 0.0), (10007, 11, 3, 1, 0.0),     # two units a stage, rows one stage ahead
    (1500, 65, 2, 2, 0.0), (1200, 128, 3, 2, 0.2), (9000, 100, 1, 2, 0.0)])
def test_narrow_tiles_against_oracle(dev, N, R, L, Hkv, dead, flags):
    s = _session(N, R, dead)
    batch = synth.make_batch(synth.Shape(L=L, Hq=4 * Hkv, Hkv=Hkv, D=128), [s], seed=N + R, kv_dtype=synth.BF16,
                             layout="paged")
    blob = synth.residual_blob(128, seed=9) if flags else None
    got = _scores(dev, batch, blob, flags, narrow=N <= 16384)
    sets = oracle.sets(batch.S(0), s.pi, s.qs, s.qe, s.C, synth.DEAD_SLOT)
    want = oracle.scores(batch.k_pool, batch.S(0), sets, batch.M_of(0), Hkv, R, blob, flags, batch.qpos_of(0),
                         synth.DEAD_SLOT)
    check_scores(got, want, sets["cand"], RESID_MFMA_FLOOR if flags else SCORE_FLOOR)


@pytest.mark.parametrize("flags", [0, ikv.IKV_RESIDUAL])
@pytest.mark.parametrize("R", [1, 4, 16, 20, 64, 90])
@pytest.mark.parametrize("N,dead", [(3001, 0.2), (12000, 0.0)])     # tiles of 32 and of 64 entries
def test_narrow_tiles_give_the_bits_of_the_wide_ones(dev, N, dead, R, flags):
    shape = synth.Shape(L=1, Hq=8, Hkv=2, D=128)
    specs = [_session(N, R, dead), _session(15500, R)]
    batch = synth.make_batch(shape, specs, seed=R, kv_dtype=synth.BF16, layout="paged")
    blob = synth.residual_blob(128, seed=9) if flags else None
    both = _scores(dev, batch, blob, flags, narrow=False)    # more than 512 groups
    first = RetentionStep(batch, dev, residual=blob, flags=flags)
    first.init_dead_slot()
    one = ikv.Sessions([{k: getattr(first.sess[0], k) for k, _ in ikv.Session._fields_}], dev)   # the first alone
    assert _narrow(_launched(lambda: ikv.score_history(first.pool, one, first.S, first.M, first.scores, first.ws,
                                                       qpos=first.qpos, residual=first.residual, flags=flags)))
    n = specs[0].N
    assert np.array_equal(first.host("scores")[:n].view(np.uint32), both[:n].view(np.uint32))
