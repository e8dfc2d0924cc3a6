"""The vector-unit residual head takes 8, 16 or 32 candidates per workgroup, by the number of
positions: scores against the float64 oracle on both sides of the two lines."""
import pytest

import oracle
import synth
from paper_2606_09916_amd import ikv
from paper_2606_09916_amd.step import RetentionStep
from parity import SCORE_FLOOR, check_scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,N", [(64, 61), (64, 4096), (64, 4103), (64, 8192), (64, 8201), (128, 900), (128, 4200),
                                 (128, 8300)])
def test_residual_candidates_per_workgroup(dev, D, N):
    s = synth.SessionSpec(N=N, C=N // 4, pi=4, qs=N - 20, qe=N, R=3, dead_frac=0.1)
    batch = synth.make_batch(synth.Shape(L=1, Hq=4, Hkv=2, D=D), [s], seed=D + N, kv_dtype=synth.F32, layout="paged")
    blob = synth.residual_blob(D, seed=7)
    st = RetentionStep(batch, dev, residual=blob, flags=ikv.IKV_RESIDUAL)
    st.init_dead_slot()
    st.score()
    sets = oracle.sets(batch.S(0), s.pi, s.qs, s.qe, s.C, synth.DEAD_SLOT)
    want = oracle.scores(batch.k_pool, batch.S(0), sets, batch.M_of(0), 2, s.R, blob, ikv.IKV_RESIDUAL,
                         batch.qpos_of(0), synth.DEAD_SLOT)
    check_scores(st.host("scores"), want, sets["cand"], SCORE_FLOOR)
