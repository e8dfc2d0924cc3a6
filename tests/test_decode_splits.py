"""How many splits a decode call gives each live list, read from the size of its workspace
(one partial state per session, layer, query head and split): every session the same number,
so that no workgroup of the grid is without work where the lists are equally long, and never a
grid that fills its rounds of 512 workgroups less than one split more or less per session
would by more than it has to."""
import pytest

from paper_2606_09916_amd import ikv

SHAPES = [(48, 40, 8, 128, ikv.IKV_BF16, 2), (36, 32, 8, 128, ikv.IKV_BF16, 2), (48, 20, 4, 128, ikv.IKV_BF16, 1),
          (28, 28, 4, 128, ikv.IKV_BF16, 1), (80, 64, 8, 128, ikv.IKV_BF16, 2), (13, 3, 3, 128, ikv.IKV_BF16, 3),
          (1, 8, 2, 64, ikv.IKV_F32, 2), (6, 8, 4, 64, ikv.IKV_BF16, 4), (2, 8, 8, 128, ikv.IKV_F32, 8)]


def _splits(shape, lists):
    """Splits per session, and units (workgroups per split of a session)."""
    L, Hq, Hkv, D, dtype, groups = shape
    pool = ikv.Pool(L, Hq, Hkv, D, 1 << 20, 0, dtype, 4096, 4096)
    rows = [dict(slot_off=0, mem_off=0, qspan_off=0, qpos_off=0, N=n, pi=0, qs=0, qe=0, C=n, radix_prefix=0, R=4, nq=0)
            for n in lists]
    n = ikv.workspace_bytes(pool, ikv.Sessions(rows, "cpu"), ikv.CALL_DECODE)
    per = len(lists) * L * Hq * (D + 2) * 4
    assert n % per == 0, "sessions of a batch have unequal splits, or workgroups without work"
    return n // per, L * groups


def _fill(n):
    return n / (-(-n // 512) * 512)


@pytest.mark.parametrize("n", [1, 63, 64, 500, 1000, 2048, 4096, 8192, 40000])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 8, 16, 64, 700])
@pytest.mark.parametrize("shape", SHAPES)
def test_equal_lists(shape, B, n):
    s, units = _splits(shape, [n] * B)
    assert 1 <= s <= min(64, -(-n // 64))
    one_round = max(1, min(512 // (units * B), 64, -(-n // 64)))
    if B == 1:
        assert s == one_round
    else:
        assert s >= one_round and _fill(s * units * B) >= _fill(one_round * units * B)
        assert s == one_round or n >= 256 * s


@pytest.mark.parametrize("lists", [(8192, 517), (12000, 4587, 9162, 1712, 6911), (3000, 300, 2000, 900, 1500),
                                   (40000,) + (64,) * 9, (700, 100), (8192, 8000, 7900)])
@pytest.mark.parametrize("shape", SHAPES)
def test_uneven_lists(shape, lists):
    s, units = _splits(shape, lists)
    wgs = units * len(lists)
    one_round = max(1, min(512 // wgs, 64, -(-max(lists) // 64)))
    assert s >= one_round
    if s > one_round:
        assert s <= 8 and max(lists) >= 256 * s and _fill(s * wgs) >= _fill(one_round * wgs)
        assert s <= 4 or (max(lists) >= 768 * s and s * wgs <= 10 * 512)
