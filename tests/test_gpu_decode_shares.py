"""Decode of several sessions of uneven live counts: every session has the same number of
splits, chosen from the bounds known on the host, so that short lists leave splits empty.
Against float64 attention; a bf16 output is at most half a unit in the last place (2^-9 of
its value) and the softmax's float32 rounding from it."""
import numpy as np
import pytest

from paper_2606_09916_amd import ikv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,L,Hkv,G,D,bound,counts", [
    ("bf16", 2, 4, 5, 128, 9000, (9000, 1, 700, 64, 0, 65, 4097)),        # an empty session
    ("bf16", 2, 2, 4, 128, 300, (2999, 3000, 17)),                        # live lists past the budget's bound
    ("bf16", 48, 4, 2, 128, 6000, (6000, 1200, 5999, 31, 4000, 2500, 3333, 100, 2)),   # seven splits, some empty
    ("bf16", 40, 1, 8, 128, 40, (40,) * 70 + (3,) * 2),                   # many sessions of one split
    ("f32", 1, 2, 4, 64, 4000, (4000, 0, 128, 129, 1000)),
    ("f32", 1, 1, 1, 64, 70, (0, 0, 0)),                                  # nothing live at all
])
def test_uneven_live_lists(dtype, L, Hkv, G, D, bound, counts):
    import torch
    dev = torch.device("cuda")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev).manual_seed(len(counts) + L)
    slots = max(max(counts), 64) + 1
    k = torch.randn(L, slots, Hkv, D, generator=gen, device=dev).to(dt)
    v = torch.randn(L, slots, Hkv, D, generator=gen, device=dev).to(dt)
    q = torch.randn(len(counts), L, Hkv * G, D, generator=gen, device=dev).to(dt)
    rows, off = [], 0
    for n in counts:
        N = max(n, 8)
        rows.append(dict(N=N, R=G, pi=0, qs=N - 4, qe=N, C=bound, radix_prefix=0, nq=0, slot_off=off, mem_off=0,
                         qspan_off=0, qpos_off=0))
        off += N
    live = torch.zeros(off, dtype=torch.int32, device=dev)
    for r, n in zip(rows, counts):
        live[r["slot_off"]:r["slot_off"] + n] = 1 + torch.randperm(slots - 1, generator=gen, device=dev)[:n].int()
    n_live = torch.tensor(counts, dtype=torch.int32, device=dev)
    out = torch.full_like(q, 7.0)
    pool = ikv.make_pool(k, v, L, Hkv * G, Hkv, D, slots, 0)
    ikv.decode_attend_slotmap(pool, ikv.Sessions(rows, dev), q, live, n_live, out, ikv.Workspace(dev))
    for b, (r, n) in enumerate(zip(rows, counts)):
        want = torch.zeros(L, Hkv, G, D, dtype=torch.float64, device=dev)
        idx = live[r["slot_off"]:r["slot_off"] + n].long()
        for l in range(L):
            if n:
                K, V = (x[l][idx].double().transpose(0, 1).contiguous() for x in (k, v))
                s = q[b, l].double().view(Hkv, G, D) @ K.transpose(1, 2).contiguous() / np.sqrt(D)
                want[l] = torch.softmax(s, dim=2) @ V
        want = want.view(L, Hkv * G, D)
        err = (out[b].double() - want).abs()
        # values are of order one: 2e-5 for the float32 sums of up to 9000 terms
        tol = 2e-5 + (want.abs() * 2.0 ** -8 if dtype == "bf16" else 0.0)
        assert bool((err <= tol).all()), f"session {b}: {float(err.max())}"
