"""The kept-position list of the compact apply path is written by one workgroup per span of
1024 positions (2048 past 65,536): the rows each destination slot receives and the count,
at the edges of the spans."""
import numpy as np
import pytest
import torch

import synth
from paper_2606_09916_amd import ikv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,frac", [(1, 1.0), (1023, 0.5), (1024, 1.0), (1025, 0.5), (5000, 0.02), (66001, 0.3),
                                    (3000, 0.0)])
def test_compact_list_spans(dev, N, frac):
    g = np.random.default_rng(N)
    D, slots = 64, 2 * N + 2
    S = (1 + g.permutation(N)).astype(np.int32)
    S[g.random(N) < 0.1] = synth.DEAD_SLOT
    keep = (g.random(N) < frac).astype(np.uint8)              # kept marks on dead positions do not count
    kept = np.nonzero((keep != 0) & (S != synth.DEAD_SLOT))[0]
    dst = np.zeros(N, np.int32)
    dst[:len(kept)] = N + 1 + g.permutation(len(kept))
    k = torch.zeros((1, slots, 1, D), device=dev)
    v = torch.from_numpy(g.standard_normal((1, slots, 1, D)).astype(np.float32)).to(dev)
    v0 = v.clone()
    pool = ikv.make_pool(k, v, 1, 1, 1, D, slots, synth.DEAD_SLOT)
    sess = ikv.Sessions([dict(slot_off=0, mem_off=0, qspan_off=0, qpos_off=0, N=N, pi=0, qs=N, qe=N, C=N, radix_prefix=0,
                              R=1, nq=0)], dev)
    n_keep = torch.full((1,), -1, dtype=torch.int32, device=dev)
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    ikv.compact_apply(pool, sess, t(S), t(keep), t(dst), n_keep, ikv.Workspace(dev))
    assert int(n_keep.item()) == len(kept)
    want = v0.clone()
    want[0, dst[:len(kept)].astype(np.int64)] = v0[0, S[kept].astype(np.int64)]
    assert torch.equal(v, want)
