"""The row copy of the compact apply path at the edges of its steps: pools whose pair groups
are fewer than a workgroup, not a multiple of the steps in flight, and more kept positions
than workgroups. Keys against the float64 rotation within the rounding of the pool's type
(half a unit in the last place of a row's pair, plus float32 products), values bit for bit."""
import numpy as np
import pytest

from paper_2606_09916_amd import ikv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,L,Hkv,D,N", [("f32", 1, 1, 64, 40), ("f32", 3, 2, 64, 700), ("f32", 9, 8, 128, 300),
                                             ("bf16", 1, 1, 64, 33), ("bf16", 36, 8, 128, 129), ("bf16", 13, 8, 128, 90),
                                             ("bf16", 2, 1, 128, 9500), ("bf16", 2, 1, 128, 12000), ("bf16", 4, 8, 128, 70),
                                             ("bf16", 5, 8, 128, 70), ("bf16", 12, 8, 128, 60),
                                             ("f32", 4, 8, 128, 50), ("f32", 17, 1, 64, 90)])
def test_compact_rows(dtype, L, Hkv, D, N):
    import torch
    dev = torch.device("cuda")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev).manual_seed(N)
    slots = 2 * N + 1
    k = torch.randn(L, slots, Hkv, D, generator=gen, device=dev).to(dt)
    v = torch.randn(L, slots, Hkv, D, generator=gen, device=dev).to(dt)
    k0, v0 = k.clone(), v.clone()
    S = 1 + torch.randperm(N, generator=gen, device=dev).int()
    keep = (torch.rand(N, generator=gen, device=dev) < 0.8).to(torch.uint8)
    kept = keep.nonzero().reshape(-1)
    dst = torch.zeros(N, dtype=torch.int32, device=dev)
    dst[:len(kept)] = N + 1 + torch.randperm(N, generator=gen, device=dev)[:len(kept)].int()
    rows = [dict(N=N, R=1, pi=0, qs=N - 4, qe=N, C=N // 2, radix_prefix=0, nq=0, slot_off=0, mem_off=0, qspan_off=0,
                 qpos_off=0)]
    n_keep = torch.zeros(1, dtype=torch.int32, device=dev)
    ikv.compact_apply(ikv.make_pool(k, v, L, Hkv, Hkv, D, slots, 0), ikv.Sessions(rows, dev), S, keep, dst, n_keep,
                      ikv.Workspace(dev), rope_base=1e4)
    assert int(n_keep[0]) == len(kept)
    src, to = S[kept].long(), dst[:len(kept)].long()
    assert torch.equal(v[:, to], v0[:, src])
    h = D // 2
    t = torch.arange(len(kept), device=dev)
    ang = (t - kept).double()[:, None] * 1e4 ** (-torch.arange(h, device=dev, dtype=torch.float64) / h)
    co, si = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = k0[:, src, :, :h].double(), k0[:, src, :, h:].double()
    want = torch.cat([a * co - b * si, b * co + a * si], dim=-1)
    size = torch.cat([a.abs() + b.abs()] * 2, dim=-1)
    tol = size * 2.0 ** -22 + (want.abs() * 2.0 ** -8 if dtype == "bf16" else 0.0)
    assert bool(((k[:, to].double() - want).abs() <= tol).all())
    rest = torch.ones(slots, dtype=torch.bool, device=dev)
    rest[to] = False
    assert torch.equal(k[:, rest], k0[:, rest]) and torch.equal(v[:, rest], v0[:, rest])
